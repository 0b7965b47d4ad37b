// Attention launches: the launch shape (workgroups, rows per workgroup)
// and the choice of kernel instantiation by head dimension, mask, LSE output
// and row-map mode.  The kernel itself is in attn_kernel.hpp.
#include <mutex>

#include "attn_kernel.hpp"

using pulsar_attn::KernelArgs;

namespace {

// Work counters of the persistent causal launches: a slot per (device,
// stream), since launches on one stream never overlap, while launches on
// different streams may.  A slot holds a counter per KV head and the count
// of finished workgroups; it is zero before and after every launch.  A
// stream beyond the slots, or one being captured into a graph (whose
// replays could run beside other launches from the same stream), gets the
// plain one-workgroup-per-item launch.
constexpr int kSchedSlots = 64;
constexpr int kSchedWords = 32;  // up to 31 KV heads
__device__ __align__(256) unsigned g_sched[kSchedSlots][kSchedWords];

struct SchedDevice {
  bool ready = false;
  unsigned* base = nullptr;  // device address of g_sched on this device
  int n_cu = 0;
  int used = 0;
  hipStream_t stream[kSchedSlots];
};
std::mutex g_sched_mu;
SchedDevice g_sched_dev[64];

// The counter slot of the current device and this stream (and the device's
// compute-unit count), or null.
unsigned* sched_slot(hipStream_t stream, int* n_cu) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)
    return nullptr;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(g_sched_mu);
  SchedDevice& sd = g_sched_dev[dev];
  if (!sd.ready) {
    void* p = nullptr;
    int cu = 0;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_sched)) != hipSuccess ||
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cu < 1)
      return nullptr;
    sd.base = static_cast<unsigned*>(p);
    sd.n_cu = cu;
    sd.ready = true;
  }
  int slot = -1;
  for (int i = 0; i < sd.used; ++i)
    if (sd.stream[i] == stream) slot = i;
  if (slot < 0) {
    if (sd.used == kSchedSlots) return nullptr;
    slot = sd.used++;
    sd.stream[slot] = stream;
  }
  *n_cu = sd.n_cu;
  return sd.base + (size_t)slot * kSchedWords;
}

}  // namespace

int attn_rows_per_wg(int group, bool causal) {
  const int heads_per_wg = group >= 4 ? 4 : group;
  const int waves = causal ? kCausalWaves : kPartialWaves;
  return 32 * kQT * (waves / heads_per_wg);
}

int launch_attention(const AttnLaunch& a, hipStream_t stream) {
  // load offsets are formed with 24-bit multiplies: a K/V row of at most
  // 2^24 bytes (and, with buffers below 2 GiB, positions below 2^24)
  if ((int64_t)a.Hkv * a.d * 2 >= (1 << 24)) return PULSAR_EUNSUPPORTED;
  KernelArgs ka;
  ka.a = a;
  ka.group = a.Hq / a.Hkv;
  ka.heads_per_wg = ka.group >= 4 ? 4 : ka.group;
  ka.hsub = ka.group / ka.heads_per_wg;
  ka.rows_per_wg = attn_rows_per_wg(ka.group, a.causal != 0);
  ka.n_row_tiles = (a.n_q + ka.rows_per_wg - 1) / ka.rows_per_wg;
  ka.nz = a.nz_kv * a.nsplit;
  ka.sched = nullptr;
  ka.grid = 0;
  int n_cu = 256;
  if (a.causal && a.Hkv < kSchedWords) {
    ka.sched = sched_slot(stream, &n_cu);
    ka.grid = n_cu;
  }
  // The key-split form, where a launch has no more items than compute units:
  // it then takes as long as its longest item, the last row tile over all
  // keys, which the split halves (and its workgroups load every tile for half
  // as many rows).  Without / with it, us: 20 items of 1280 rows, 4 / 1 heads of
  // 64 34.3 / 24.5; 128 of 512 rows (two sequences), 32 / 8 heads of 128 32.4 /
  // 29.0; 256 of 4096 rows, 16 / 4 heads of 128 116 / 90; 256 of 2048 rows, 32 /
  // 32 heads of 128 62.7 / 51.5.  With more items the queue balances them: 384 of
  // 2851 rows, 16 / 16 heads of 64 88 / 101, 424 of 3380 rows, 32 / 8 of 128 120
  // / 150.  So it does, over half a compute unit each, where items are short: a
  // workgroup of several heads has 64 or 128 rows, and up to 2048 keys of them
  // are split only while the halves fit the chip at once (160 items of 640 rows,
  // 64 / 2 heads of 64 22.1 / 28.6; 192 of 1024 rows, 24 / 2 of 128, two sequences
  // 39.5 / 42.2; 256 of 2048 rows, 32 / 8 of 128 67.9 / 71.7; 176 of 2816 rows, 16
  // / 4 of 128 77.6 / 56.2), or are few for their length and read few KV heads
  // (160 of 1280 rows, 32 / 2 of 128 43.9 / 38.2).  At d 64 a short row's tiles
  // are not worth the merge (128 of 256 rows, 64 / 2 heads, two sequences 15.4 /
  // 18.5).
  const int64_t items = (int64_t)ka.n_row_tiles * ka.hsub * a.Hkv * ka.nz;
  const bool all = ka.heads_per_wg == 1 || a.n_kv > 2048 ||
                   (a.d == 128 && a.Hkv * ka.nz <= 4 && items * 8 <= a.n_kv);
  const int64_t most = all ? n_cu : ka.heads_per_wg == 4 && a.d == 64 && a.n_kv < 512 ? n_cu / 4
                                                                                     : n_cu / 2;
  const int64_t split_lds = a.d == 128 ? attn_lds<128>(true, a.map.n_runs)
                                       : attn_lds<64>(true, a.map.n_runs);
  ka.ksplit = a.causal && items <= most && a.n_kv >= 256 && split_lds + 16 <= PULSAR_LDS_BYTES;
  if (ka.ksplit) {
    ka.rows_per_wg /= 2;
    ka.n_row_tiles = (a.n_q + ka.rows_per_wg - 1) / ka.rows_per_wg;
  }
  const bool lse = a.lse != nullptr;
  if (a.d == 128) return pulsar_attn::launch_d128(ka, a.causal != 0, lse, a.map.mode, stream);
  return pulsar_attn::launch_d64(ka, a.causal != 0, lse, a.map.mode, stream);
}
