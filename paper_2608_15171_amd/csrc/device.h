// Host-side helpers shared by the entry points: kernel launchers and the
// current device's properties.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.h"

namespace ppas {

struct DeviceInfo {
  bool known = false;
  bool gfx950 = false;
  int cus = 256;
};

// Compute-unit count and architecture of the current device (cached per device).
// Without a usable device: 256 CUs, not gfx950.
DeviceInfo current_device();

// The packed attention launch and, when n_comb > 0, the split-merge launch.
hipError_t launch_attn_step(const uint16_t* q, uint16_t* out, const uint16_t* kp, const uint16_t* vp,
                            const int32_t* bt, int32_t bt_stride, int32_t hq, int32_t hkv, float scale,
                            const WorkItem* items, int n_items, const CombineItem* comb, int n_comb,
                            float2* part_ml, float* part_acc, int tile_pos, hipStream_t stream,
                            hipEvent_t ev_start, hipEvent_t ev_stop, hipEvent_t ev_merge_start,
                            hipEvent_t ev_merge_stop);

// The gate-up projection: y = x w^T (hidden a multiple of 64), or with `act` the
// gated activation of its two halves, y[t][f] = silu(s[t][f]) s[t][N2/2 + f]
// (N2 even, y [T][N2/2]). The reduction is split over at most max_splits
// workgroups per output tile, as many as pay, whose fp32 partial sums
// (gateup_workspace_bytes of `part`, columns in weight-row order) a second launch
// adds in order. `cus` is the device's compute-unit count. gateup_choose (host
// only) is the kernel that such a call takes; `aligned`: x and w on 16 bytes.
struct GateupChoice {
  enum Kernel { kTiles = 0, kRows = 1, kGeneral = 2 };
  Kernel kernel = kGeneral;
  int32_t rows = 256;                       // token rows of a main tile (64: none), or of a few-row workgroup
  int32_t g = 0, wr = 0;                    // few rows: weight-row tiles per workgroup and their rows
  int32_t splits = 1;
  int32_t main_m = 0, tail_m = 0;           // tiles: main ones along the token rows, 64-row ones after them
  int32_t light = 0, grid = 0, block = 8;   // tiles: see GemmArgs
};
GateupChoice gateup_choose(int32_t T, int32_t H, int32_t N2, bool act, bool aligned, int max_splits, int cus);
hipError_t launch_gateup(const uint16_t* x, const uint16_t* w, uint16_t* y, int32_t T, int32_t H, int32_t N2,
                         bool act, int max_splits, float* part, int cus, hipStream_t stream, hipEvent_t ev_start,
                         hipEvent_t ev_stop);
// The projection's kernel for operands the regular one does not take (not 16-byte
// aligned, or rows too long for its offsets): the partials when splits > 1.
hipError_t launch_gateup_any(const uint16_t* x, const uint16_t* w, uint16_t* y, int32_t T, int32_t H, int32_t N2,
                             bool act, int splits, float* part, int cus, hipStream_t stream, hipEvent_t ev_start,
                             hipEvent_t ev_stop);
// Output tiles of a call: 256 x 256, plus 64 x 256 for the last T % 256 token rows.
int64_t gateup_tiles(int32_t T, int32_t N2);
// The most reduction splits a call on a device with `cus` compute units uses (1: none).
int gateup_splits(int32_t T, int32_t H, int32_t N2, int cus);
size_t gateup_workspace_bytes(int32_t T, int32_t N2, int splits);

// XOR of every 16-byte word of buf (bytes a multiple of 16) into sink[0..3],
// read once by a streaming grid of up to `cus` workgroups.
hipError_t launch_stream_read(const void* buf, size_t bytes, uint32_t* sink, int cus, hipStream_t stream,
                              hipEvent_t ev_start, hipEvent_t ev_stop);

}  // namespace ppas
