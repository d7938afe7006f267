// Internal launch interface between the C ABI layer and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace vitattn {

// Workgroups of a kernel that the current device holds at once, and its CUs;
// zeros if the runtime cannot say. Looked up once per device (no stream work,
// so a graph capture may hold it).
struct Resident {
  int workgroups, cus;
};
class ResidentCache {
 public:
  Resident get(const void* kernel, int threads) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return {0, 0};
    long long known = known_[dev].load(std::memory_order_relaxed);
    if (known == 0) {
      int per_cu = 0, cus = 0;
      known = -1;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) == hipSuccess &&
          hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && per_cu * cus > 0)
        known = (long long)cus << 32 | (per_cu * cus);
      known_[dev].store(known, std::memory_order_relaxed);
    }
    return known > 0 ? Resident{(int)(known & 0x7fffffff), (int)(known >> 32)} : Resident{0, 0};
  }

 private:
  static constexpr int kDevices = 64;
  std::atomic<long long> known_[kDevices] = {};  // 0 = not looked up, -1 = unknown
};

// Estimated time of a forward or dQ launch of `nw` waves (32 nw query rows)
// per workgroup, in units of one round of 8-wave workgroups, one per CU:
// whole rounds, then the last one by how many workgroups a CU gets, and the
// start and end of each workgroup, worth so many 64-key tiles. Only 4-wave
// workgroups share a CU, and then one's start and end overlap another's tiles.
// Without the device's figures 8 waves win.
inline double launch_cost(int BH, int Nq, int Nk, int nw, const Resident& r) {
  if (r.workgroups <= 0) return nw == 8 ? 0. : 1.;
  const long long n = (long long)BH * ((Nq + 32 * nw - 1) / (32 * nw));
  const long long rounds = n / r.workgroups, left = n - rounds * r.workgroups;
  const double tiles = (Nk + 63) / 64, alone = 1. + 6. / tiles;
  if (nw != 4) return (double)(rounds + (left > 0)) * (nw / 8.) * alone;
  // 1 .. 3 per CU: measured 0.66-0.86, 1.02-1.05, 1.48-1.52; the ends 3-4.6
  // tiles' time with company, 6-7 alone (N = 512 .. 16,384, every width)
  constexpr double of[4] = {0., 0.86, 1.04, 1.5};
  const int per_cu = r.workgroups / r.cus < 3 ? r.workgroups / r.cus : 3;
  const int last = (int)((left + r.cus - 1) / r.cus);
  return (rounds * of[per_cu] + of[last < per_cu ? last : per_cu]) * (per_cu > 1 ? 1. + 4.5 / tiles : alone);
}

// Where the rows of one [B][H][N][d] operand live: element strides of the
// batch, head and row dimensions (the d elements of a row are contiguous).
struct Map {
  long long sb, sh;
  int ld;
  __host__ __device__ long long head(int bh, int H) const { return (bh / H) * sb + (bh % H) * sh; }
};
inline Map dense_map(int H, int N, int d) { return Map{(long long)H * N * d, (long long)N * d, d}; }

// Tile width of the attention kernels for head dim d (a multiple of 8, at
// most 160): columns d .. D-1 of every tile are zeros.
inline int tile_width(int d) { return d <= 64 ? 64 : d <= 96 ? 96 : d <= 128 ? 128 : 160; }

struct FwdArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  float* o;
  float* lse;  // [B][H][Nq], dense
  Map mq, mk, mv, mo;
  int H, BH, Nq, Nk, d;  // query rows and key rows per (b, h); d the head dim
  float scale;
  hipStream_t stream;
};

struct BwdArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const float* o;
  const uint16_t* dout;
  const float* lse;  // [B][H][Nq], dense
  float* dq;
  float* dk;
  float* dv;
  float* drow;  // workspace region 0: D = rowsum(dO o O), [BH][Nq]
  float* lse2;  // workspace region 1: LSE * log2(e), [BH][Nq]
  uint16_t* ds;  // dS mode: workspace region 2 (the dS blocks), else nullptr
  Map mq, mk, mv, mo, mg, mdq, mdk, mdv;  // mg: dout
  int H, BH, Nq, Nk, d;  // query rows and key rows per (b, h); d the head dim
  float scale;
  bool accumulate_dq;  // dq += this call's dQ instead of dq = ...
  // training step: an fp32 upstream gradient, which the row-dot pass rounds
  // into dout_w (= dout, dense), and bf16 outputs
  const float* grad;
  Map mgrad;
  uint16_t* dout_w;
  bool dq16, kv16;  // dq, and dk and dv (only where dkdv_one_sum), are bf16
  hipStream_t stream;
};

struct MergeArgs {
  const float* o_parts;    // [P][BH][N][d]
  const float* lse_parts;  // [P][BH][N]
  float* o;                // [BH][N][d]
  float* lse;              // [BH][N]
  int P, BH, N, d;
  hipStream_t stream;
};

hipError_t launch_fwd(const FwdArgs& a);
int fwd_waves(const FwdArgs& a);  // waves per workgroup of the forward that launch_fwd takes

// Workspace layout of the backward pass: two fp32 regions of region_floats
// each (D, then LSE*log2(e)), every region 256-byte aligned; in the dS mode a
// third region holds the dS blocks: 2 KB per 32 keys x 32 queries of every
// head, key blocks rounded up to the dK/dV kernel's 128 keys (its 64-key form
// covers as many) and query blocks to its 64-query tiles.
inline size_t bwd_region_floats(long long rows) { return (size_t)((rows + 63) / 64) * 64; }
inline int ds_key_blocks(int Nk) { return (Nk + 127) / 128 * 4; }
inline int ds_query_blocks(int Nq) { return (Nq + 63) / 64 * 2; }
inline size_t ds_region_bytes(long long BH, int Nq, int Nk) {
  return (size_t)BH * ds_key_blocks(Nk) * ds_query_blocks(Nq) * 2048;
}

// Backward stages; launch_bwd runs all three in order.
hipError_t launch_bwd_rowdot(const BwdArgs& a);
hipError_t launch_bwd_dkdv(const BwdArgs& a);
hipError_t launch_bwd_dq(const BwdArgs& a);  // dQ from stored dS when a.ds is set
hipError_t launch_bwd(const BwdArgs& a);
// The forms that launch_bwd takes: keys per dK/dV workgroup, its whole key
// blocks and those split over two workgroups, the 64-key workgroups launched
// behind them; waves per dQ workgroup.
struct BwdForms {
  int dkdv_keys, dkdv_whole, dkdv_split, dkdv_rest64, dq_waves;
};
BwdForms bwd_forms(const BwdArgs& a);
bool dkdv_one_sum(int Nq);  // every key block sums its query tiles as one sum (never as two added in memory)
hipError_t launch_merge(const MergeArgs& a);

// Ulysses layout copies (see vitattn_ulysses.hip for the row orders)
enum { kUlyssesPack = 0, kUlyssesUnpack = 1, kUlyssesPackOut = 2, kUlyssesUnpackOut = 3 };
struct UlyssesArgs {
  const void* src;
  void* dst;
  int B, Nl, H, P, row_bytes, mode;
  hipStream_t stream;
};
hipError_t launch_ulysses(const UlyssesArgs& a);
long ulysses_blocks(int Nl, int H, int row_bytes);  // grid.x of the layout kernels

// Channel aggregation (attention of one learnable query per head over the C
// channel tokens of each of M patches); see vitattn_agg.hip.
constexpr int kAggChunkGroup = 12;  // 1 KB chunks of a [C][d] block whose loads one wave issues together
struct AggArgs {
  const uint16_t* q;     // [H][d]
  const uint16_t* k;     // [M][H][C][d]
  const uint16_t* v;     // [M][H][C][d]
  const float* o;        // [M][H][d]      (backward input)
  const uint16_t* dout;  // [M][H][d]
  float* o_out;          // forward output
  const float* lse;      // [M][H]         (backward input)
  float* lse_out;        // forward output
  float* dq;             // [H][d]
  float* dk;             // [M][H][C][d]
  float* dv;             // [M][H][C][d]
  float* partial;        // workspace: [agg_partials(M)][H][d]
  int M, H, C, d;
  float scale;
  hipStream_t stream;
};
int agg_partials(int M);  // dq partials of the backward pass
hipError_t launch_agg_fwd(const AggArgs& a);
hipError_t launch_agg_bwd(const AggArgs& a);

}  // namespace vitattn
