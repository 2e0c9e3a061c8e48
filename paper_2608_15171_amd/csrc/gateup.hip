// Fused gate-up projection of a decoder block's MLP on gfx950 (CDNA4):
//   Y[T][N2] = X[T][H] * W[N2][H]^T
// bf16 inputs, fp32 accumulation on 16x16x32 MFMAs, output rounded to bf16
// (nearest even). W stacks the gate rows over the up rows, so one launch
// computes both projections of a prefill chunk.
//
// What bounds it: with operands of ordinary values the chip lowers its clock
// under matrix work (32x32x16 MFMAs from registers reach 1.83 PFLOP/s, 16x16x32
// 2.07, both 2.45 on zeros), so the smaller instruction is used, and everything
// beside the MFMAs has to run under them.
//
// Schedule. A workgroup of eight waves (two per SIMD) owns an output tile; the
// reduction advances 64 features per stage. Waves 0-3 and 4-7 (one of each per
// SIMD) run half a phase apart: while one half issues a phase's MFMAs, the other
// issues its transfers and operand reads for its next phase, and a workgroup
// barrier swaps the roles. Each operand of a stage is copied into LDS in units
// (half of the tile's W rows, half or all of its X rows) by 16-byte
// global-to-LDS transfers of eight whole 128-byte row runs (one cache line per
// row), and a unit's buffer is refilled two phases after it was read, so that
// transfers stay in flight across several phases and no wait drains them. The
// transfers take buffer descriptors held in scalar registers (rows past the
// edge read as zero) and one 32-bit lane offset; the stage offset is scalar.
// In LDS a row keeps its eight 16-byte chunks in an XOR-swizzled order, so an
// operand fragment (16 rows x 64 bytes) is one conflict-free ds_read_b128.
// The stream of transfers runs on into the workgroup's next tile, so a tile's
// epilogue overlaps the next tile's loads.
//   16,384 tokens, the MLP's two projections: 1,948 -> 1,640 us in turn on one card
//   (before: 32x32x16 MFMAs, one barrier and one drain of the transfers per stage);
//   2,048 x 22,016 alone 1,052-1,100 us (1.34-1.40 PFLOP/s), 11,008 x 2,048 489-511
//   us (1.45-1.51 PFLOP/s)
// (transfers issued after the operand reads 1-2 % slower, one of two among the
// MFMAs 4 %, both 8 %; 32x32x16 MFMAs in the same schedule 6-8 %)
//
// The MFMA's first operand is W (rows = output columns), its second X (rows =
// tokens): lane L of a 16 x 16 result then holds token row L % 16 and four
// consecutive output columns 4 (L / 16) + 0..3, which the epilogue packs into
// 8-byte LDS writes of a wave-private area; the wave's block then leaves LDS as
// row runs of 16-byte stores.
//
// Tile order. The grid holds one workgroup per compute unit, each looping over
// its tiles. Workgroup b runs on XCD b % 8; each XCD takes a contiguous range
// of tiles, and tiles are numbered in groups of 8 token-row tiles that share a
// weight tile, so the workgroups resident on one XCD share operand tiles in
// that XCD's L2.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "device.h"
#include "gateup_device.h"

namespace ppas {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBN = 256;                 // output columns per tile
constexpr int kHN = kBN / 2;             // rows of a W unit
constexpr int kBK = 64;                  // features per stage
constexpr int kRow = 2 * kBK;            // bytes of a row in a stage
constexpr int kTailBM = 64;              // token rows per small tile
constexpr int kGroupM = 8;               // token-row tiles per tile-order group
constexpr int kSmem = 160 * 1024;        // the LDS of one compute unit
constexpr int64_t kMaxPitch = int64_t(1) << 24;   // 256 rows of fewer bytes than this fit a 32-bit offset

struct GemmArgs {
  const uint16_t* x;
  const uint16_t* w;
  uint16_t* y;
  float* part;            // splits > 1: fp32 partial sums [splits][T][N2]
  int32_t T, H, N2;
  int32_t I;              // with the gated activation: N2 / 2 intermediate features
  int32_t tiles_n;        // 256-column tiles
  int32_t main_m;         // main tiles along the token rows
  int32_t tail_m;         // 64-row tiles of the rows after them
  int32_t splits;         // reduction split over this many workgroups per tile
  int32_t light;          // small tiles a workgroup with one main tile fewer takes first
  int32_t block;          // stages per block of a two-level sum (tiles below 256 rows, few-row calls): 4 or 8
};

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return uint32_t(__builtin_amdgcn_readfirstlane(int(v))); }

// One output tile over stages k_lo .. k_hi - 1 of reduction split `split`.
struct Item {
  int m0, n0, split, k_lo, k_hi;
};

// Position u of a list of tiles x splits -> tile. The first 8 * (n / 8) positions
// give XCD u % 8 the contiguous range xcd * (n / 8) + u / 8 (workgroup b runs on
// XCD b % 8, and the grid is a multiple of 8 whenever it is smaller than the list);
// the remainder runs in order. Entry v is tile v % tiles of split v / tiles.
__device__ __forceinline__ Item item_at(const GemmArgs& a, int u, int tiles_m, int bm, int m_first) {
  Item r;
  const int ntiles = tiles_m * a.tiles_n;
  const int per_xcd = ntiles * a.splits / 8;
  const int v = (u < 8 * per_xcd) ? (u % 8) * per_xcd + u / 8 : u;
  const int t = v % ntiles;
  r.split = v / ntiles;
  const int nk = a.H / kBK, kq = nk / a.splits, kr = nk - kq * a.splits;
  r.k_lo = r.split * kq + min(r.split, kr);
  r.k_hi = r.k_lo + kq + (r.split < kr);
  const int first_m = t / (kGroupM * a.tiles_n) * kGroupM;
  const int gm = min(kGroupM, tiles_m - first_m);
  const int in_grp = t - first_m * a.tiles_n;
  r.m0 = m_first + (first_m + in_grp % gm) * bm;
  r.n0 = (in_grp / gm) * kBN;
  return r;
}

// The main tiles of workgroup b: positions b, b + grid, ...
struct MainList {
  int at, n;
  __device__ __forceinline__ MainList(const GemmArgs& a) {
    n = a.main_m * a.tiles_n * a.splits;
    at = blockIdx.x;
  }
  __device__ __forceinline__ bool more() const { return at < n; }
  __device__ __forceinline__ void next() { at += gridDim.x; }
};

// The small tiles of workgroup b. When the main tiles do not divide evenly, the
// last grid - rem workgroups have one main tile fewer; each of these takes
// `light` small tiles first (about the time of a main tile), and the rest are
// dealt to all workgroups in turn.
struct SmallList {
  int at, n, in_light, nlight;
  __device__ __forceinline__ SmallList(const GemmArgs& a) {
    const int grid = gridDim.x, b = blockIdx.x;
    n = a.tail_m * a.tiles_n * a.splits;
    const int rem = (a.main_m * a.tiles_n * a.splits) % grid;
    nlight = grid - rem;
    in_light = min(int64_t(n), int64_t(a.light) * nlight);
    at = b - rem;
    if (at < 0 || at >= in_light) at = in_light + b;
  }
  __device__ __forceinline__ bool more() const { return at < n; }
  __device__ __forceinline__ void next() {
    if (at < in_light) {
      at += nlight;
      if (at >= in_light) at = in_light + blockIdx.x;
    } else {
      at += gridDim.x;
    }
  }
};

// Buffer descriptor of up to `rows` rows of a row-major matrix from row r0 on
// (rows past the matrix are out of range: they read as zero), in scalar registers.
struct Rows {
  uint32_t lo, hi, bytes;
  __device__ __forceinline__ void set(const uint16_t* p, int r0, int rows_total, int rows, int H) {
    const int valid = max(0, min(rows, rows_total - r0));
    const uint64_t b = reinterpret_cast<uint64_t>(p + size_t(valid > 0 ? r0 : 0) * H);
    lo = uniform(uint32_t(b));
    hi = uniform(uint32_t(b >> 32));
    bytes = uniform(uint32_t(valid) * uint32_t(H) * 2);
  }
};

#ifdef __HIP_DEVICE_COMPILE__
// 16 bytes per lane from the rows into LDS: lane L lands at lds + 16 L.
__device__ __forceinline__ void transfer(const Rows& r, char* lds, uint32_t lane_off, uint32_t stage_off) {
  const uint64_t b = uint64_t(uniform(r.lo)) | (uint64_t(uniform(r.hi)) << 32);
  __amdgpu_buffer_rsrc_t d =
      __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, int(uniform(r.bytes)), 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(d, (lds_void*)lds, 16, lane_off, uniform(stage_off), 0, 0);
}
#endif

// A tile of BM token rows x 256 columns as the waves see it. The W rows of a stage
// are two units (with the activation: the gate rows and the up rows of 128
// features); with BM = 256 the X rows are two units as well (four phases per
// stage, one per pair of units, and a ring of two stages), below that one (two
// phases, three stages). Wave (wn, wm) owns, of every unit pair, QN columns x QM
// token rows as kNT x kMT MFMA tiles.
template <int BM>
struct Tile {
  static constexpr int XH = BM == 256 ? 2 : 1;             // X units
  static constexpr int WNW = BM == 256 ? 2 : 4;            // waves along the columns
  static constexpr int HM = BM / XH;                       // rows of an X unit
  static constexpr int QN = kHN / WNW, QM = HM / (kWaves / WNW);
  static constexpr int kNT = QN / 16, kMT = QM / 16;
  static constexpr int kRing = BM == 256 ? 2 : 3;
  static constexpr bool kTwoLevel = BM != 256;             // block sums added to a running total
  static constexpr int kStage = (kBN + BM) * kRow;
  static constexpr int kOffX = kBN * kRow;
  static constexpr int kDW = kHN / 8 / kWaves, kDX = HM / 8 / kWaves;   // transfers per wave and unit
  static constexpr int kEpiRows = QN == 64 ? QM : 32;      // rows staged at a time in the epilogue
  static constexpr int kEpi = QN * kEpiRows * 2;           // a wave's staging bytes
  static_assert(kRing * kStage + kWaves * kEpi <= kSmem, "the ring and the staging areas fit");
  static_assert(kDW * 8 * kWaves == kHN && kDX * 8 * kWaves == HM && kDX >= 1, "whole transfers per wave");
  static_assert(QM % kEpiRows == 0 && kEpiRows % 16 == 0, "whole staged blocks");
};

// A wave's kEpiRows x QN block of bf16 results, staged in LDS by `put` in an
// XOR-swizzled order, to rows m.. and columns n.. of y (T rows, `cols` columns).
template <int QN, int ROWS>
struct Staged {
  static constexpr int kLPR = QN / 8, kRPI = 64 / kLPR, kIt = ROWS / kRPI;
  static constexpr int kShift = kLPR == 8 ? 1 : 2;   // rows that share a 256-byte bank run
  __device__ static __forceinline__ void put(char* eb, int row, int col, float v0, float v1, float v2, float v3) {
    u32x2 v;
    v[0] = pack_bf16x2(v0, v1);
    v[1] = pack_bf16x2(v2, v3);
    *reinterpret_cast<u32x2*>(eb + row * QN * 2 + 16 * ((col >> 3) ^ ((row >> kShift) & (kLPR - 1))) +
                              2 * (col & 7)) = v;
  }
  __device__ static __forceinline__ void out(const char* eb, int lane, uint16_t* y, int m, int n, int T, int cols) {
    u32x4 v[kIt];
#pragma unroll
    for (int i = 0; i < kIt; ++i) v[i] = lds16(eb + 1024 * i + 16 * lane);
#pragma unroll
    for (int i = 0; i < kIt; ++i) {
      const int row = i * kRPI + lane / kLPR;
      const int c = n + 8 * ((lane % kLPR) ^ ((row >> kShift) & (kLPR - 1)));
      if (m + row >= T) continue;
      uint16_t* dst = y + size_t(m + row) * cols + c;
      if (c + 8 <= cols) {
        *reinterpret_cast<u32x4*>(dst) = v[i];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (c + e < cols) dst[e] = uint16_t(v[i][e >> 1] >> (16 * (e & 1)));
      }
    }
  }
};

// Every tile of this workgroup's list, in turn.
template <int BM, bool kAct, typename List>
__device__ __forceinline__ void run_tiles(const GemmArgs& a, char* smem, int m_first, int tiles_m) {
#ifdef __HIP_DEVICE_COMPILE__
  using C = Tile<BM>;
  constexpr int QN = C::QN, QM = C::QM, kNT = C::kNT, kMT = C::kMT;
  List todo(a);
  if (!todo.more()) return;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool late = w >= kWaves / 2;   // the half that runs half a phase behind
  const int wn = w % C::WNW, wm = w / C::WNW;

  // Transfers. One covers eight rows of a unit: lane L lands at row L / 8, position
  // L % 8, and fetches the chunk stored there under the swizzle (row R keeps chunk
  // c at c ^ (R / 2) % 8). Stage `dk` of the list's tile `ahead` goes to ring slot
  // `dslot`.
  uint32_t vw[C::kDW], vx[C::kDX];
  {
    auto lane_off = [&](int r) {
      return uint32_t(r) * (uint32_t(a.H) * 2) + 16 * ((lane & 7) ^ ((r >> 1) & 7));
    };
#pragma unroll
    for (int i = 0; i < C::kDW; ++i) vw[i] = lane_off((w * C::kDW + i) * 8 + lane / 8);
#pragma unroll
    for (int i = 0; i < C::kDX; ++i) vx[i] = lane_off((w * C::kDX + i) * 8 + lane / 8);
  }
  Rows rw[2], rx[C::XH];
  List ahead(a);
  int dk, dk_hi, dslot = 0;
  auto aim = [&]() {
    const Item it = item_at(a, ahead.at, tiles_m, BM, m_first);
    if (kAct) {
      rw[0].set(a.w, it.n0 / 2, a.I, kHN, a.H);
      rw[1].set(a.w + size_t(a.I) * a.H, it.n0 / 2, a.I, kHN, a.H);
    } else {
      rw[0].set(a.w, it.n0, a.N2, kHN, a.H);
      rw[1].set(a.w, it.n0 + kHN, a.N2, kHN, a.H);
    }
#pragma unroll
    for (int g = 0; g < C::XH; ++g) rx[g].set(a.x, it.m0 + g * C::HM, a.T, C::HM, a.H);
    dk = it.k_lo;
    dk_hi = it.k_hi;
  };
  aim();
  auto issue_w = [&](int h) {
#pragma unroll
    for (int i = 0; i < C::kDW; ++i)
      transfer(rw[h], smem + dslot * C::kStage + h * kHN * kRow + (w * C::kDW + i) * 1024, vw[i], dk * kRow);
  };
  auto issue_x = [&](int g) {
#pragma unroll
    for (int i = 0; i < C::kDX; ++i)
      transfer(rx[g], smem + dslot * C::kStage + C::kOffX + g * C::HM * kRow + (w * C::kDX + i) * 1024, vx[i],
               dk * kRow);
  };
  auto next_stage = [&]() {
    dslot = dslot + 1 == C::kRing ? 0 : dslot + 1;
    if (++dk == dk_hi) {
      List n = ahead;
      n.next();
      if (n.more()) {
        ahead = n;
        aim();
      } else {
        // past the last tile: its last stage again, into slots that nobody reads
        // (the waits count transfers, so their number stays the same)
        --dk;
      }
    }
  };

  // Operand fragments: (row tile t, 32-feature step j) of lane L is row 16 t + L % 16,
  // chunk 4 j + L / 16; the swizzle term depends on the lane only.
  int aw[2], ax[2], rslot = 0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = lane & 15;
    const int o = r * kRow + 16 * ((4 * j + (lane >> 4)) ^ ((r >> 1) & 7));
    aw[j] = wn * QN * kRow + o;
    ax[j] = C::kOffX + wm * QM * kRow + o;
  }
  bf16x8 fw[2][kNT][2], fx[C::XH][kMT][2];
  f32x4 acc[2][C::XH][kNT][kMT];
  auto read_w = [&](int h) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < kNT; ++t) fw[h][t][j] = as_bf16x8(lds16(smem + aw[j] + (h * kHN + 16 * t) * kRow));
  };
  auto read_x = [&](int g) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < kMT; ++t) fx[g][t][j] = as_bf16x8(lds16(smem + ax[j] + (g * C::HM + 16 * t) * kRow));
  };
  auto next_slot = [&]() {
    const int step = rslot + 1 == C::kRing ? -(C::kRing - 1) * C::kStage : C::kStage;
    rslot = rslot + 1 == C::kRing ? 0 : rslot + 1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      aw[j] += step;
      ax[j] += step;
    }
  };
  // The MFMAs of one phase; the first stage of a tile starts the sums from zero.
  auto mma = [&](int h, int g, bool first) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int tj = 0; tj < kMT; ++tj)
#pragma unroll
        for (int ti = 0; ti < kNT; ++ti) {
          const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
          acc[h][g][ti][tj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fw[h][ti][j], fx[g][tj][j], (first && j == 0) ? zero : acc[h][g][ti][tj], 0, 0, 0);
        }
  };

  // One stage. BM = 256, phases (W unit, X unit): (0,0) (0,1) (1,1) (1,0). The
  // memory slots read X 0; X 1; W 1; W 0 of the next stage, and issue W 1 of the
  // stage after next; then W 0, X 0, X 1 of the one after that: each unit two
  // phases after its buffer was last read, and five units behind the one the next
  // phase needs. A phase's MFMAs wait for what its memory slot read, except W 0, which
  // the next stage uses first: the last phase waits for it by itself. BM < 256, phases
  // W 0 and W 1: the slots read X and W 0; W 1, and issue X and W 0, then W 1, two
  // stages ahead of the reads.
  auto stage = [&](bool first) {
    if constexpr (BM == 256) {
      constexpr int kWaitA = 3 * C::kDX + 2 * C::kDW, kWaitB = 2 * C::kDX + 3 * C::kDW;
      issue_w(1);
      __builtin_amdgcn_sched_barrier(0);
      read_x(0);
      wait_vmcnt<kWaitB>();
      bare_barrier();
      mma(0, 0, first);
      bare_barrier();
      next_stage();
      issue_w(0);
      __builtin_amdgcn_sched_barrier(0);
      read_x(1);
      wait_vmcnt<kWaitB>();
      bare_barrier();
      mma(0, 1, first);
      bare_barrier();
      issue_x(0);
      __builtin_amdgcn_sched_barrier(0);
      read_w(1);
      wait_vmcnt<kWaitA>();
      bare_barrier();
      mma(1, 1, first);
      bare_barrier();
      issue_x(1);
      __builtin_amdgcn_sched_barrier(0);
      next_slot();
      read_w(0);
      wait_vmcnt<kWaitA>();
      bare_barrier();
      mma(1, 0, first);
      // these MFMAs don't use the W 0 just read: it is waited for here, a barrier before
      // the other half may refill its buffer
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);
    } else {
      issue_x(0);
      issue_w(0);
      __builtin_amdgcn_sched_barrier(0);
      read_x(0);
      read_w(0);
      wait_vmcnt<2 * (C::kDX + C::kDW) + C::kDW>();
      bare_barrier();
      mma(0, 0, first);
      bare_barrier();
      issue_w(1);
      __builtin_amdgcn_sched_barrier(0);
      read_w(1);
      next_slot();
      wait_vmcnt<C::kDX + 3 * C::kDW>();
      bare_barrier();
      mma(1, 0, first);
      next_stage();
    }
  };

  if constexpr (BM == 256) {
    issue_w(0);
    issue_x(0);
    issue_x(1);
    issue_w(1);
    next_stage();
    issue_w(0);
    issue_x(0);
    issue_x(1);
    wait_vmcnt<3 * C::kDX + 2 * C::kDW>();   // W 0 and X 0 of the first stage have landed
    bare_barrier();
    read_w(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);      // W 0 is read before its buffer may be refilled
    bare_barrier();
  } else {
    for (int s = 0; s < 2; ++s) {
      issue_x(0);
      issue_w(0);
      issue_w(1);
      next_stage();
    }
    wait_vmcnt<C::kDX + 3 * C::kDW>();       // X and W 0 of the first stage have landed
    bare_barrier();
  }
  if (late) bare_barrier();

  for (; todo.more(); todo.next()) {
    const Item it = item_at(a, todo.at, tiles_m, BM, m_first);
    // Below 256 rows the sums are kept in two levels, blocks of a.block stages added
    // to a running total: one chain over 2,048 features rounds 1.6 times as far off as
    // eight partial sums (blocks of eight stages cost 2-4 % of a tile, of four 3-9 %).
    f32x4 total[2][C::XH][kNT][kMT];
    if (C::kTwoLevel) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int ti = 0; ti < kNT; ++ti)
#pragma unroll
          for (int tj = 0; tj < kMT; ++tj) total[h][0][ti][tj] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int k = it.k_lo; k < it.k_hi;) {
      const int k_end = C::kTwoLevel ? min(k + a.block, it.k_hi) : it.k_hi;
      if (k > it.k_lo) bare_barrier();
      stage(true);
      for (++k; k < k_end; ++k) {
        bare_barrier();
        stage(false);
      }
      if (C::kTwoLevel) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int ti = 0; ti < kNT; ++ti)
#pragma unroll
            for (int tj = 0; tj < kMT; ++tj)
              total[h][0][ti][tj] += acc[h][0][ti][tj];
      }
    }
    const auto& sum = C::kTwoLevel ? total : acc;
    // Results, in the MFMA slot of the last phase: element r of sum[h][g][ti][tj] is
    // token row 16 tj + L % 16 of the wave's rows of X unit g, column 16 ti + 4 (L / 16)
    // + r of its columns of W unit h.
    if (a.splits > 1) {
      float* pb = a.part + size_t(it.split) * a.T * a.N2;
#pragma unroll
      for (int g = 0; g < C::XH; ++g)
#pragma unroll
        for (int tj = 0; tj < kMT; ++tj) {
          const int m = it.m0 + g * C::HM + wm * QM + 16 * tj + (lane & 15);
          if (m >= a.T) continue;
          float* row = pb + size_t(m) * a.N2;
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ti = 0; ti < kNT; ++ti) {
              const int c = wn * QN + 16 * ti + 4 * (lane >> 4);
              if (kAct) {
                // partials keep the weight-row order: gate feature f at column f, its up
                // row at I + f (features from I on belong to neither)
                const int f = it.n0 / 2 + c;
                if (f < a.I) store_part(row + h * a.I, f, a.I, (a.I & 3) == 0, sum[h][g][ti][tj]);
              } else {
                store_part(row, it.n0 + h * kHN + c, a.N2, (a.N2 & 3) == 0, sum[h][g][ti][tj]);
              }
            }
        }
    } else {
      char* eb = smem + C::kRing * C::kStage + w * C::kEpi;
      using S = Staged<QN, C::kEpiRows>;
      constexpr int kTB = C::kEpiRows / 16;   // row tiles staged at a time
      const int ncols = kAct ? a.I : a.N2;
#pragma unroll
      for (int h = 0; h < (kAct ? 1 : 2); ++h)
#pragma unroll
        for (int g = 0; g < C::XH; ++g)
#pragma unroll
          for (int tb = 0; tb < kMT; tb += kTB) {
#pragma unroll
            for (int tj = 0; tj < kTB; ++tj)
#pragma unroll
              for (int ti = 0; ti < kNT; ++ti) {
                const f32x4 v = sum[h][g][ti][tb + tj];
                const int row = 16 * tj + (lane & 15), col = 16 * ti + 4 * (lane >> 4);
                if constexpr (kAct) {
                  const f32x4 u = sum[1][g][ti][tb + tj];
                  S::put(eb, row, col, silu_f32(v[0]) * u[0], silu_f32(v[1]) * u[1], silu_f32(v[2]) * u[2],
                         silu_f32(v[3]) * u[3]);
                } else {
                  S::put(eb, row, col, v[0], v[1], v[2], v[3]);
                }
              }
            S::out(eb, lane, a.y, it.m0 + g * C::HM + wm * QM + 16 * tb,
                   (kAct ? it.n0 / 2 : it.n0 + h * kHN) + wn * QN, a.T, ncols);
          }
      __builtin_amdgcn_s_waitcnt(0xC07F);   // the reads of rows past the edge, which no store waits for
    }
    bare_barrier();
  }
  if (!late) bare_barrier();
  wait_vmcnt<0>();   // no transfer outlives its buffers
  bare_barrier();
#endif
}

// Main tiles of BM token rows (256 or 128; none when main_m is 0), then the 64-row
// tiles of the rows after them.
template <int BM, bool kAct>
__global__ __launch_bounds__(kThreads, 1) void gateup_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[kSmem];
  run_tiles<BM, kAct, MainList>(a, smem, 0, a.main_m);
  run_tiles<kTailBM, kAct, SmallList>(a, smem, a.main_m * BM, a.tail_m);
}

// Few token rows (decode iterations): the weights are streamed once and the rest
// has to stay out of the way. A workgroup owns G tiles of WR weight rows (with
// the activation half of them gate rows, half the up rows of the same features)
// x 16 XT token rows, and its waves split the reduction between them in
// 64-feature chunks, so that no operand is shared between waves: each runs a ring
// of its own in LDS, kSlots chunks deep, with no barrier until the end and up to
// 160 KB of a compute unit's LDS in flight. (Loads straight into the MFMA operand
// registers take twice the time: adjacent lanes then read different rows, and the
// address unit takes one lane per clock instead of four. Eight waves measured
// 0-10 % slower than four.) At the end the waves' sums meet in LDS and are added
// in order. Against one tile kernel with a split reduction and its reducing launch,
// calls one after another, weights from memory: 24 tokens x 2,048 x 22,016 with the
// activation 28.4 -> 22.7 us (4.0 TB/s of weights), 11,008 x 2,048 24.6 -> 17.5 us (X,
// read by every workgroup, bounds it), 2,048 x 2,048 11.8 -> 8.6 us, of which 4.3 are
// the kernel's (12.5 before); 1 token 25.7 -> 21.5, 22.7 -> 13.4, 10.9 -> 8.4 us.
constexpr int kRowsWaves = 4;

template <int XT, int G, int WR, bool kAct>
__global__ __launch_bounds__(64 * kRowsWaves, 1) void gateup_rows_kernel(GemmArgs a) {
  constexpr int NW = kRowsWaves;
  constexpr int kSlot = (G * WR + XT * 16) * kRow;        // bytes of a chunk
  constexpr int kMoves = (G * WR + XT * 16) / 8;          // its transfers
  // With one weight-row tile the block sums of up to kOrdered blocks are kept beside
  // the rings and added in order; otherwise the waves' totals take the rings' place.
  constexpr int kOrdered = G == 1 ? 8 : 0;
  constexpr int kSumBytes = (G == 1 ? kOrdered : NW) * G * XT * 1024;
  constexpr int kRoom = kSmem - (G == 1 ? kSumBytes : 0);
  constexpr int kSlots = kRoom / NW / kSlot < 4 ? kRoom / NW / kSlot : 4;
  constexpr int kRings = NW * kSlots * kSlot;
  constexpr int kBytes = G == 1 ? kRings + kSumBytes : kRings > kSumBytes ? kRings : kSumBytes;
  static_assert(kSlots >= 2 && kBytes <= kSmem, "at least two chunks per wave; the sums fit");
  static_assert(!kAct || G % 2 == 0, "gate and up rows in pairs");
  __shared__ __attribute__((aligned(1024))) char smem[kBytes];
#ifdef __HIP_DEVICE_COMPILE__
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int m0 = blockIdx.y * 16 * XT;
  const int c0 = blockIdx.x * (kAct ? WR / 2 : WR) * G;   // first column (feature) of the tile
  constexpr int kGP = kAct ? G / 2 : G;                   // weight-row tiles per weight half
  const int ncols = kAct ? a.I : a.N2;

  Rows rw[2], rx;
  rw[0].set(a.w, c0, ncols, WR * kGP, a.H);
  rw[1].set(a.w + (kAct ? size_t(a.I) * a.H : 0), c0, ncols, WR * kGP, a.H);
  rx.set(a.x, m0, a.T, 16 * XT, a.H);
  const uint32_t pitch = uint32_t(a.H) * 2;
  // transfer i of a tile: rows 8 i + L / 8, swizzled as in the tile kernels
  uint32_t off[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 8 * i + lane / 8;
    off[i] = uint32_t(r) * pitch + 16 * ((lane & 7) ^ ((r >> 1) & 7));
  }
  const int nchunks = a.H / kBK;
  char* ring = smem + w * kSlots * kSlot;
  auto load = [&](int slot, int c) {
    char* dst = ring + slot * kSlot;
    const uint32_t so = uint32_t(c) * kRow;
#pragma unroll
    for (int t = 0; t < XT; ++t)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        transfer(rx, dst + t * 16 * kRow + i * 1024, off[i] + uint32_t(16 * t) * pitch, so);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int i = 0; i < WR / 8; ++i)
        transfer(rw[g / kGP], dst + (XT * 16 + g * WR) * kRow + i * 1024, off[i] + uint32_t(WR * (g % kGP)) * pitch, so);
  };
  // a tile of eight weight rows fills the MFMA's 16 twice; the second half is dropped
  int frag_x[2], frag_w[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = r16 % WR;
    frag_x[j] = r16 * kRow + 16 * ((4 * j + q) ^ ((r16 >> 1) & 7));
    frag_w[j] = r * kRow + 16 * ((4 * j + q) ^ ((r >> 1) & 7));
  }

  // Two-level sums, as in the tile kernels. In order: blocks of four chunks, wave w
  // taking blocks w, w + NW, ...; otherwise blocks of eight of the wave's chunks
  // w, w + NW, ... (or of four, a.block)
  f32x4 acc[G][XT], total[G][XT];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int t = 0; t < XT; ++t) total[g][t] = acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4* sums = reinterpret_cast<f32x4*>(smem + (G == 1 ? kRings : 0));   // [blocks or waves][G * XT][64]
  const int nblocks = (nchunks + 3) / 4;
  const bool ordered = nblocks <= kOrdered;
  auto end_block = [&](int blk) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < XT; ++t) {
        if (ordered)
          sums[(blk * G * XT + g * XT + t) * 64 + lane] = acc[g][t];
        else
          total[g][t] += acc[g][t];
        acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  // the i-th chunk of this wave; neighbouring chunks are read together where the
  // order allows it (2-3 us faster on wide outputs)
  auto chunk_of = [&](int i) { return ordered ? 4 * (w + NW * (i >> 2)) + (i & 3) : w + NW * i; };
  int n = w < nchunks ? (nchunks - 1 - w) / NW + 1 : 0;                    // chunks of this wave
  if (ordered) {
    const int mine = w < nblocks ? (nblocks - 1 - w) / NW + 1 : 0;
    // only the last block of all may be short
    n = mine == 0 ? 0 : 4 * mine - ((w + NW * (mine - 1) == nblocks - 1) ? 4 * nblocks - nchunks : 0);
  }
  if (n > 0) {
    const int last = (ordered ? 4 : a.block) - 1;
    // past its last chunk a wave fetches that one again, so that every wait counts
    // the same number of younger transfers
#pragma unroll
    for (int s = 0; s < kSlots; ++s) load(s, chunk_of(min(s, n - 1)));
    int slot = 0;
    for (int i = 0; i < n; ++i) {
      wait_vmcnt<kMoves * (kSlots - 1)>();
      asm volatile("" ::: "memory");
      const char* src = ring + slot * kSlot;
      bf16x8 fx[XT][2], fw[G][2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int t = 0; t < XT; ++t) fx[t][j] = as_bf16x8(lds16(src + t * 16 * kRow + frag_x[j]));
#pragma unroll
        for (int g = 0; g < G; ++g) fw[g][j] = as_bf16x8(lds16(src + (XT * 16 + g * WR) * kRow + frag_w[j]));
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // the chunk is in registers before its slot is refilled
      asm volatile("" ::: "memory");
      load(slot, chunk_of(min(i + kSlots, n - 1)));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < XT; ++t)
#pragma unroll
          for (int g = 0; g < G; ++g)
            acc[g][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[g][j], fx[t][j], acc[g][t], 0, 0, 0);
      slot = slot + 1 == kSlots ? 0 : slot + 1;
      if ((i & last) == last || i + 1 == n) end_block(w + NW * (i >> 2));
    }
  }
  wait_vmcnt<0>();
  if (G > 1) __syncthreads();               // every ring is idle before the sums take its place
  if (!ordered) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < XT; ++t) sums[(w * G * XT + g * XT + t) * 64 + lane] = total[g][t];
  }
  __syncthreads();
  const int nsums = ordered ? nblocks : NW;
  // wave w finishes results w, w + NW, ...: lane L holds token row L % 16, columns
  // 4 (L / 16) .. + 3
  for (int f = w; f < kGP * XT; f += NW) {
    f32x4 s = sums[f * 64 + lane];
    for (int v = 1; v < nsums; ++v) s += sums[(v * G * XT + f) * 64 + lane];
    if constexpr (kAct) {
      f32x4 u = sums[(kGP * XT + f) * 64 + lane];
      for (int v = 1; v < nsums; ++v) u += sums[(v * G * XT + kGP * XT + f) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = silu_f32(s[e]) * u[e];
    }
    const int m = m0 + 16 * (f % XT) + r16, c = c0 + WR * (f / XT) + 4 * q;
    if (m >= a.T || 4 * q >= WR) continue;
    uint16_t* dst = a.y + size_t(m) * ncols + c;
    if (c + 4 <= ncols) {
      u32x2 v;
      v[0] = pack_bf16x2(s[0], s[1]);
      v[1] = pack_bf16x2(s[2], s[3]);
      *reinterpret_cast<u32x2*>(dst) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < ncols) dst[e] = uint16_t(pack_bf16x2(s[e], 0.f) & 0xffff);
    }
  }
#endif
}

// Token rows per workgroup.
int rows_tokens(int32_t T) { return T <= 16 ? 16 : T <= 32 ? 32 : 64; }

template <int G, int WR, bool kAct>
void launch_rows(const GemmArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int ncols = kAct ? a.I : a.N2, per = (kAct ? WR / 2 : WR) * G;
  const int xt = rows_tokens(a.T) / 16;
  const dim3 grid(unsigned((ncols + per - 1) / per), unsigned((a.T + 16 * xt - 1) / (16 * xt))), block(64 * kRowsWaves);
  if (xt == 1)
    hipExtLaunchKernelGGL((gateup_rows_kernel<1, G, WR, kAct>), grid, block, 0, stream, ev_start, ev_stop, 0, a);
  else if (xt == 2)
    hipExtLaunchKernelGGL((gateup_rows_kernel<2, G, WR, kAct>), grid, block, 0, stream, ev_start, ev_stop, 0, a);
  else
    hipExtLaunchKernelGGL((gateup_rows_kernel<4, G, WR, kAct>), grid, block, 0, stream, ev_start, ev_stop, 0, a);
}

// y = bf16(sum over splits of the partials), the splits summed in order; thread i
// covers elements 4i .. 4i + 3 of the flattened [T][N2] output.
__global__ __launch_bounds__(256) void gateup_reduce_kernel(const float* part, uint16_t* y, int64_t total,
                                                            int32_t splits) {
  const int64_t e0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (e0 >= total) return;
  if (e0 + 4 <= total) {
    f32x4 s = *reinterpret_cast<const f32x4*>(part + e0);
    for (int k = 1; k < splits; ++k) s += *reinterpret_cast<const f32x4*>(part + size_t(k) * total + e0);
    u32x2 v;
    v[0] = pack_bf16x2(s[0], s[1]);
    v[1] = pack_bf16x2(s[2], s[3]);
    *reinterpret_cast<u32x2*>(y + e0) = v;
  } else {
    for (int64_t e = e0; e < total; ++e) {
      float s = part[e];
      for (int k = 1; k < splits; ++k) s += part[size_t(k) * total + e];
      y[e] = uint16_t(pack_bf16x2(s, 0.f) & 0xffff);
    }
  }
}

// The gated activation from split partials: z[m][f] = bf16(silu(g) * u), g and u
// the in-order sums over splits of partial columns f and I + f of row m. Thread i
// covers elements 4i .. 4i + 3 of the flattened [T][I] output.
__global__ __launch_bounds__(256) void gateup_act_reduce_kernel(const float* part, uint16_t* y, int32_t T,
                                                                int32_t I, int32_t splits) {
  const int64_t total = int64_t(T) * I;
  const int64_t e0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (e0 >= total) return;
  const int64_t plane = int64_t(T) * 2 * I;   // one split's [T][2I] partials
  auto one = [&](int64_t e) {
    const int64_t m = e / I, f = e % I;
    const float* pg = part + m * 2 * I + f;
    float g = pg[0], u = pg[I];
    for (int k = 1; k < splits; ++k) {
      g += pg[size_t(k) * plane];
      u += pg[size_t(k) * plane + I];
    }
    return silu_f32(g) * u;
  };
  if ((I & 3) == 0 && e0 + 4 <= total) {
    const int64_t m = e0 / I, f = e0 % I;
    const float* pg = part + m * 2 * I + f;
    f32x4 g = *reinterpret_cast<const f32x4*>(pg), u = *reinterpret_cast<const f32x4*>(pg + I);
    for (int k = 1; k < splits; ++k) {
      g += *reinterpret_cast<const f32x4*>(pg + size_t(k) * plane);
      u += *reinterpret_cast<const f32x4*>(pg + size_t(k) * plane + I);
    }
    u32x2 v;
    v[0] = pack_bf16x2(silu_f32(g[0]) * u[0], silu_f32(g[1]) * u[1]);
    v[1] = pack_bf16x2(silu_f32(g[2]) * u[2], silu_f32(g[3]) * u[3]);
    *reinterpret_cast<u32x2*>(y + e0) = v;
  } else {
    for (int64_t e = e0; e < e0 + 4 && e < total; ++e) y[e] = uint16_t(pack_bf16x2(one(e), 0.f) & 0xffff);
  }
}

}  // namespace

namespace {

// How a call is tiled and split.
struct Shape {
  int bm = 0;               // main tiles of 256 or 128 rows; 64: small tiles only
  int splits = 1;
  int32_t main_m = 0, tail_m = 0, light = 0;
  int64_t items = 0;
  double cost = 0;
};

// Microseconds of one stage and, beside the stages, of one tile, by tile rows; of
// the reducing launch, for each split (its chain of loads), and of its partial sums'
// bytes; and the share by which a full chip slows every stage. Fitted to 520 timed
// calls (64 to 8,200 tokens, the decoder layer's four projections, every tile shape
// and split; 8 % rms), over which the choice made with them is 0.8 % slower than the
// best one on average. kWeightBytes, the rate that the weights come in no faster than,
// and kReduceSplit (more rows hide the chain) belong to the fit at rows_cost.
constexpr double kStage256 = 0.92, kStage128 = 0.66, kStage64 = 0.53;
constexpr double kTile256 = 5.3, kTile128 = 1.4, kTile64 = 0.4;
constexpr double kReduce = 4.25, kReduceSplit = 0.12, kPartBytes = 5.5e6, kLoaded = 0.186, kWeightBytes = 9.45e6;

constexpr int kRowsMaxT = 256;   // the few-row kernel measured up to here; from about 64 rows the tiles win on wide outputs

Shape shape_cost(int32_t T, int32_t H, int32_t N2, int grid_max, int bm, int splits) {
  Shape s;
  s.bm = bm;
  s.splits = splits;
  const int64_t tiles_n = (N2 + kBN - 1) / kBN;
  s.main_m = bm == kTailBM ? 0 : T / bm;
  const int64_t rest = T - int64_t(s.main_m) * bm;
  s.tail_m = int32_t((rest + kTailBM - 1) / kTailBM);
  const int64_t nf = s.main_m * tiles_n * splits, ns = s.tail_m * tiles_n * splits;
  s.items = nf + ns;
  const double nk = double(H / kBK) / splits;
  const double cf = bm == 256 ? nk * kStage256 + kTile256 : nk * kStage128 + kTile128;
  const double cs = nk * kStage64 + kTile64;
  s.light = std::max(0, int(cf / cs));
  const int64_t grid = std::min<int64_t>(s.items, grid_max);
  const int64_t rem = nf % grid, light = grid - rem;
  const int64_t in_light = std::min<int64_t>(ns, s.light * light);
  const int64_t extra = (ns - in_light + grid - 1) / grid;
  const double t_light = double(nf / grid) * cf + double((in_light + light - 1) / light + extra) * cs;
  const double t_heavy = rem ? double(nf / grid + 1) * cf + double(extra) * cs : 0;
  s.cost = std::max(std::max(t_light, t_heavy) * (1 + kLoaded * std::min(1.0, double(s.items) / grid_max)),
                    2.0 * N2 * H / kWeightBytes);
  if (splits > 1) s.cost += kReduce + (T <= kRowsMaxT ? kReduceSplit * splits : 0) + 2.0 * splits * double(T) * N2 * 4 / kPartBytes;
  return s;
}

// The few-row kernel's variants: weight-row tiles per workgroup and their rows.
// One eight-row tile doubles the workgroups where the columns are few.
struct RowsShape {
  int g, wr;
  bool with_act, without;
};
constexpr RowsShape kRowsShapes[] = {{1, 8, false, true}, {1, 16, false, true}, {2, 8, true, false},
                                     {2, 16, true, true}, {4, 16, true, true},  {6, 16, true, true}};

// Microseconds: the weights stream at 8 TB/s over the chip or 56 GB/s into one compute
// unit, X (from L2) at 99 GB/s, one after the other; every round of resident workgroups
// takes 2.8 us to fill; the rest is the launch and the final sums. Where variants come
// out alike, more workgroups of fewer weight-row tiles have more loads in flight: 8,192
// x 8,192 with one token 30.0 us in one tile against 32.9 in two. Fitted with
// kTilesBase, the launches of a call of the tile kernels, to 14,500 timed calls (60
// projections, 1 to 1,000 tokens, every variant, the weights from memory: none is read
// again before 640 MB of others; 15 % rms, the tiles 14 %). The choice is then 1.5 %
// slower than the best on average. Constants fitted to weights that a repeated call
// finds in the 256 MB cache made it 3.6 %, and some calls slower than one tile kernel
// for all sizes had been: 11,008 x 512 with 48 tokens 24.2 us where that one takes 22.3
// (now 18.9), 16,384 x 8,192 with 16 tokens 82.4 against 73.8 (now 65.2).
constexpr double kTilesBase = 4.64;
double rows_cost(int32_t T, int32_t H, int32_t N2, int cus, const RowsShape& v) {
  const int xt = rows_tokens(T) / 16;
  const double cols = double((int64_t(N2) + v.g * v.wr - 1) / (v.g * v.wr));
  const double mt = (T + 16 * xt - 1) / (16 * xt);
  const int slot = (v.g * v.wr + 16 * xt) * kRow;
  const int ring = 4 * slot * std::min(4, kSmem / 4 / slot);
  const int per_cu = std::max(1, kSmem / std::max(ring, 4 * v.g * xt * 1024));
  const double wgs = cols * mt, room = double(cus) * per_cu;
  const double rounds = wgs > room ? std::ceil(wgs / room) * per_cu : std::max(1.0, wgs / cus);
  const double w = 2.0 * v.g * v.wr * H, x = 2.0 * T / mt * H;
  const double cost = 2.9 + std::max(rounds * w / 5.57e4, mt * 2.0 * N2 * H / 8.0e6) + rounds * x / 9.93e4 +
                      0.02 * v.g * xt + 2.84 * std::ceil(wgs / room);
  return cost * (1 + 0.01 * (v.g - 1));
}

}  // namespace

int64_t gateup_tiles(int32_t T, int32_t N2) {
  return (int64_t(T / 256) + (T % 256 + kTailBM - 1) / kTailBM) * ((N2 + kBN - 1) / kBN);
}

int gateup_splits(int32_t T, int32_t H, int32_t N2, int cus) {
  const int64_t tiles = gateup_tiles(T, N2);
  const int nk = H / kBK;
  if (tiles <= 0 || tiles >= cus) return 1;
  // about one workgroup per compute unit, each with at least four stages
  return int(std::max<int64_t>(1, std::min<int64_t>(cus / tiles, nk / 4)));
}

size_t gateup_workspace_bytes(int32_t T, int32_t N2, int splits) {
  return splits > 1 ? size_t(splits) * size_t(T) * size_t(N2) * sizeof(float) : 0;
}

GateupChoice gateup_choose(int32_t T, int32_t H, int32_t N2, bool act, bool aligned, int max_splits, int cus) {
  GateupChoice r;
  r.splits = max_splits;
  // The transfers need 16-byte aligned rows and 32-bit offsets within a unit.
  if (!aligned || int64_t(H) * 2 >= kMaxPitch) return r;
  // one workgroup per compute unit (a multiple of 8, so that each stays on one XCD's
  // share of the tiles)
  const int grid_max = std::max(8, cus / 8 * 8);
  // Narrow outputs (the K and V projections, whose results are cached) are summed in
  // 256-feature blocks added in order, where the hidden size is up to eight whole such
  // blocks: by blocks of four stages, or by a split into exactly these blocks. The
  // result then does not depend on the number of tokens beside it or on the workspace.
  // Other outputs, longer narrow ones among them, take the cheapest split: 2,056 x 4,096
  // x 512 takes 41.6 us unsplit, 24.0 us in three splits.
  const bool narrow = !act && N2 <= 2 * kBN && H % (4 * kBK) == 0 && H <= 8 * 4 * kBK;
  // A choice of fewer splits than allowed makes no fp32 chain longer than the most
  // splits would (`longest` stages): 256-row tiles, which keep one chain, take them all,
  // and the others sum by blocks of four stages where eight would be longer.
  const int longest = (H / kBK + max_splits - 1) / max_splits;
  Shape best;
  for (int bm : {256, 128, 64}) {
    if (bm > kTailBM && T < bm) continue;   // no tile of that height
    for (int s = 1; s <= max_splits; ++s) {
      if (bm == 256 && s < max_splits) continue;
      if (narrow && ((s > 1 && s * 4 * kBK != H) || bm == 256)) continue;
      const Shape c = shape_cost(T, H, N2, grid_max, bm, s);
      if (c.items > INT32_MAX / 2) continue;
      if (best.bm == 0 || c.cost < best.cost) best = c;
    }
  }
  if (best.bm == 0) return r;
  r.kernel = GateupChoice::kTiles;
  r.rows = best.bm;
  r.splits = best.splits;
  r.main_m = best.main_m;
  r.tail_m = best.tail_m;
  r.light = best.light;
  r.grid = int32_t(std::min<int64_t>(best.items, grid_max));
  r.block = narrow || longest < 8 ? 4 : 8;
  if (T > kRowsMaxT) return r;
  double cost = best.cost + kTilesBase;
  for (const RowsShape& v : kRowsShapes) {
    if (!(act ? v.with_act : v.without) || N2 / (v.g * v.wr) >= (1 << 22) || (narrow && v.g > 1)) continue;
    const double c = rows_cost(T, H, N2, grid_max, v);
    if (c < cost) {
      cost = c;
      r.kernel = GateupChoice::kRows;
      r.rows = rows_tokens(T);
      r.splits = 1;
      r.g = v.g;
      r.wr = v.wr;
    }
  }
  return r;
}

hipError_t launch_gateup(const uint16_t* x, const uint16_t* w, uint16_t* y, int32_t T, int32_t H, int32_t N2,
                         bool act, int max_splits, float* part, int cus, hipStream_t stream, hipEvent_t ev_start,
                         hipEvent_t ev_stop) {
  if (T <= 0) return hipSuccess;
  if (max_splits < 1 || max_splits > H / kBK || (max_splits > 1 && !part) || (act && N2 % 2 != 0))
    return hipErrorInvalidValue;
  const bool aligned = reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0;
  const GateupChoice c = gateup_choose(T, H, N2, act, aligned, max_splits, cus);
  const int splits = c.splits;
  hipEvent_t ev = splits > 1 ? nullptr : ev_stop;
  hipError_t e;
  if (c.kernel == GateupChoice::kGeneral) {
    e = launch_gateup_any(x, w, y, T, H, N2, act, splits, part, cus, stream, ev_start, ev);
  } else {
    GemmArgs a;
    a.x = x;
    a.w = w;
    a.y = y;
    a.part = part;
    a.T = T;
    a.H = H;
    a.N2 = N2;
    a.I = N2 / 2;
    // with the activation a tile holds 128 features and their two weight rows each
    a.tiles_n = (N2 + kBN - 1) / kBN;
    a.main_m = c.main_m;
    a.tail_m = c.tail_m;
    a.splits = splits;
    a.light = c.light;
    a.block = c.block;
    if (c.kernel == GateupChoice::kRows) {
      const int shape = 100 * int(act) + 10 * c.g + (c.wr == 16);
      switch (shape) {
        case 10: launch_rows<1, 8, false>(a, stream, ev_start, ev); break;
        case 11: launch_rows<1, 16, false>(a, stream, ev_start, ev); break;
        case 21: launch_rows<2, 16, false>(a, stream, ev_start, ev); break;
        case 41: launch_rows<4, 16, false>(a, stream, ev_start, ev); break;
        case 61: launch_rows<6, 16, false>(a, stream, ev_start, ev); break;
        case 120: launch_rows<2, 8, true>(a, stream, ev_start, ev); break;
        case 121: launch_rows<2, 16, true>(a, stream, ev_start, ev); break;
        case 141: launch_rows<4, 16, true>(a, stream, ev_start, ev); break;
        case 161: launch_rows<6, 16, true>(a, stream, ev_start, ev); break;
        default: return hipErrorInvalidValue;
      }
    } else {
      const dim3 grid{unsigned(c.grid)};
      if (c.rows == 256) {
        if (act)
          hipExtLaunchKernelGGL((gateup_kernel<256, true>), grid, dim3(kThreads), 0, stream, ev_start, ev, 0, a);
        else
          hipExtLaunchKernelGGL((gateup_kernel<256, false>), grid, dim3(kThreads), 0, stream, ev_start, ev, 0, a);
      } else {
        if (act)
          hipExtLaunchKernelGGL((gateup_kernel<128, true>), grid, dim3(kThreads), 0, stream, ev_start, ev, 0, a);
        else
          hipExtLaunchKernelGGL((gateup_kernel<128, false>), grid, dim3(kThreads), 0, stream, ev_start, ev, 0, a);
      }
    }
    e = hipGetLastError();
  }
  if (e != hipSuccess || splits == 1) return e;
  const int64_t total = act ? int64_t(T) * (N2 / 2) : int64_t(T) * N2;
  const int64_t blocks = (total + 1023) / 1024;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  if (act)
    hipExtLaunchKernelGGL(gateup_act_reduce_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, nullptr, ev_stop,
                          0, static_cast<const float*>(part), y, T, N2 / 2, splits);
  else
    hipExtLaunchKernelGGL(gateup_reduce_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, nullptr, ev_stop, 0,
                          static_cast<const float*>(part), y, total, splits);
  return hipGetLastError();
}

}  // namespace ppas
