// Load path: stored blobs in pinned host memory -> device staging slots -> decode, with the copy of
// group g + 1 overlapping the decode of group g (the paper charges a stored entry size / Bandwidth
// of loading delay plus its decompression overhead; Design section, utility and estimator).
//
// Consecutive blobs are packed into groups that fill one staging slot.  A group is moved by ONE
// launch of a small copy kernel that reads the pinned host memory over the bus (the blobs of a
// group need not be contiguous on the host) and also writes the group's decode descriptors at the
// head of the slot, then decoded by ONE batched decode launch; a run's last group is kept small.  Per-blob runtime copies were
// measured to leave 30-60 us of idle bus between two copies on this platform; with groups the
// fixed costs are paid once per slot.  Two streams (copy, caller's compute) and two events per slot
// order the ring; one more event orders a run's copies after what the caller's stream already holds.
#include <mutex>
#include <new>

#include "kvh_common.hpp"

namespace kvh {
namespace {

constexpr int kMaxSlots = 64;
constexpr int kMaxGroup = 32;                                   // blobs per group
constexpr size_t kDescBytes = (size_t)kMaxGroup * sizeof(kvh_kept_item);  // descriptor area at the head of a slot
constexpr int kCopyThreads = 256;
constexpr int kCopyUnroll = 4;                                  // 16-byte loads in flight per thread
constexpr uint64_t kTileWords = kCopyThreads * kCopyUnroll;     // 16-byte words of a tile: 16 KiB
// Blocks of a copy.  They have to fill the bus (57 GB/s) and not hold up the decodes that run beside the copy, whose arguments and
// packets lie in host memory behind the same bus.  Runs of several groups of 4 blobs, 16 / 48 blocks, against 4 blocks for each blob (which
// left the bus at 50 GB/s on blobs of mixed sizes, because the last and largest had 4 blocks alone): groups of 0.7 to 5 MB 1.00 to 1.03 / 0.94 to
// 1.01 times as fast (32 blobs of 0.37 MB 351 and 378 us), 5.5 to 12 MB 1.00 to 1.04 / 1.00 to 1.03, 12 to 25 MB 1.01 to 1.05 / 1.01 to 1.06, larger
// ones 1.02 to 1.06 / 1.02 to 1.06, 48 ahead by 0.3 % on average; runs of one group the same within 1 %.  24 and 32 blocks are slower than
// either in every run of several groups (0.80 to 0.96), 12, 20 and 64 by up to 2 %.
constexpr uint32_t kCopyBlocks = 48, kCopyBlocksSmall = 16;
constexpr uint32_t kSmallTiles = (12u << 20) / (kTileWords * 16);  // of a group that is copied by the fewer ones

typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

struct CopyGroup {
  int n;
  uint32_t tiles;                   // of the group
  uint32_t tile_end[kMaxGroup];     // tiles up to the end of each blob; all ones beyond the last one
  struct {
    const uint8_t* src;             // pinned host memory, device-visible
    uint64_t off, n16;              // byte offset inside the slot, size in 16-byte words
    uint64_t first;                 // its first tile
  } blob[kMaxGroup];
  kvh_kept_item item[kMaxGroup];    // decode descriptors (blob = slot + off)
};

// Block b copies tiles b, b + gridDim.x - 1, ... of the group; the last block writes the descriptors.
__global__ __launch_bounds__(kCopyThreads) void load_group_kernel(CopyGroup g, uint8_t* slot) {
  const uint32_t stride = gridDim.x - 1;
  if (blockIdx.x == stride) {
    constexpr uint32_t kWords = sizeof(kvh_kept_item) / 4;
    const uint32_t* d = reinterpret_cast<const uint32_t*>(&g.item[0]);
    for (uint32_t i = threadIdx.x; i < (uint32_t)g.n * kWords; i += kCopyThreads) reinterpret_cast<uint32_t*>(slot)[i] = d[i];
    return;
  }
  for (uint32_t t = blockIdx.x; t < g.tiles; t += stride) {
    int j = 0;
#pragma unroll
    for (int i = 0; i < kMaxGroup - 1; ++i) j += t >= g.tile_end[i] ? 1 : 0;
    const auto& b = g.blob[j];
    const uintx4* src = reinterpret_cast<const uintx4*>(b.src);
    uintx4* dst = reinterpret_cast<uintx4*>(slot + b.off);
    const uint64_t n16 = b.n16, first = (t - b.first) * kTileWords + threadIdx.x;
    uintx4 r[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u)
      if (first + u * kCopyThreads < n16) r[u] = __builtin_nontemporal_load(src + first + u * kCopyThreads);
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u)
      if (first + u * kCopyThreads < n16) dst[first + u * kCopyThreads] = r[u];
  }
}

int launch_copy(const CopyGroup& g, uint8_t* slot, hipStream_t stream) {
  const uint32_t most = g.tiles <= kSmallTiles ? kCopyBlocksSmall : kCopyBlocks;
  const uint32_t blocks = g.tiles < most ? g.tiles : most;
  hipLaunchKernelGGL(load_group_kernel, dim3(blocks + 1), dim3(kCopyThreads), 0, stream, g, slot);
  KVH_HIP_CHECK_LAUNCH();
  return KVH_OK;
}

// Everything kvh_loader_run and kvh_load_static check before they enqueue anything.  `capacity` = bytes a slot
// offers to blobs.
int validate_load(const kvh_load_item* items, int n_items, kvh_dtype dt, int l, int c, const kvh_kv_view* dst,
                  int block_tokens, size_t capacity) {
  if (items == nullptr || n_items < 1 || (dt != KVH_F16 && dt != KVH_BF16) || block_tokens < 1) return KVH_E_ARG;
  if (dst == nullptr || dst->k == nullptr || dst->v == nullptr || dst->layer_stride < 0 || dst->token_stride < c)
    return KVH_E_ARG;
  if (((reinterpret_cast<uintptr_t>(dst->k) | reinterpret_cast<uintptr_t>(dst->v)) & 15u) != 0 ||
      dst->layer_stride % 8 != 0 || dst->token_stride % 8 != 0)
    return KVH_E_ALIGN;
  for (int i = 0; i < n_items; ++i) {
    const kvh_load_item& it = items[i];
    if (it.blob_host == nullptr || it.dst_token0 < 0) return KVH_E_ARG;
    if ((reinterpret_cast<uintptr_t>(it.blob_host) & 15u) != 0) return KVH_E_ALIGN;
    if (level_bits(it.level) < 0) return KVH_E_LEVEL;
    const size_t need = kvh_blob_size(l, it.n_tokens, c, it.level);
    if (need == 0) return KVH_E_SHAPE;
    if (need > capacity) return KVH_E_SIZE;
    // the copy kernel reads the blob in place: both ends must lie in host memory the device can see
    const uint8_t* ends[2] = {static_cast<const uint8_t*>(it.blob_host), static_cast<const uint8_t*>(it.blob_host) + need - 1};
    for (const uint8_t* p : ends) {
      hipPointerAttribute_t at{};
      if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeHost) {
        (void)hipGetLastError();
        return KVH_E_ARG;
      }
    }
    if ((it.orig_tokens | it.sink | it.window) != 0) {  // a token-dropped blob: n_tokens is what is kept
      if (kvh_kept_tokens(it.orig_tokens, it.sink, it.window) != it.n_tokens) return KVH_E_SHAPE;
    }
    const int64_t span = (it.orig_tokens > it.n_tokens && !it.compact) ? it.orig_tokens : it.n_tokens;
    if (it.dst_token0 + span > INT32_MAX) return KVH_E_ARG;
  }
  return KVH_OK;
}

// Pack consecutive blobs, starting at items[first], into one slot of `capacity` bytes for blobs; returns how many
// went in (at least one: every blob has been checked against the capacity), their largest token count and whether all are raw.
int pack_group(const kvh_load_item* items, int first, int n_items, int l, int c, uint8_t* slot, size_t capacity,
               CopyGroup& g, int& max_tokens, bool& raw) {
  size_t used = 0;
  max_tokens = 0;
  raw = true;
  g.n = 0;
  g.tiles = 0;
  for (uint32_t& end : g.tile_end) end = 0xffffffffu;
  while (first + g.n < n_items && g.n < kMaxGroup) {
    const kvh_load_item& it = items[first + g.n];
    const size_t bytes = kvh_blob_size(l, it.n_tokens, c, it.level);
    if (used + bytes > capacity) break;
    g.blob[g.n] = {static_cast<const uint8_t*>(it.blob_host), kDescBytes + used, bytes / 16, g.tiles};
    g.tiles += (uint32_t)((bytes / 16 + kTileWords - 1) / kTileWords);
    g.tile_end[g.n] = g.tiles;
    g.item[g.n] = kvh_kept_item{slot + kDescBytes + used, it.n_tokens, it.level, it.dst_token0, it.page_table,
                                it.orig_tokens, it.sink, it.window, it.compact};
    if (it.n_tokens > max_tokens) max_tokens = it.n_tokens;
    raw = raw && it.level == kRawLevel;
    used += bytes;
    ++g.n;
  }
  return g.n;
}

bool fits_one_group(const kvh_load_item* items, int first, int n_items, int l, int c, size_t capacity) {
  if (n_items - first > kMaxGroup) return false;
  size_t used = 0;
  for (int i = first; i < n_items && used <= capacity; ++i) used += kvh_blob_size(l, items[i].n_tokens, c, items[i].level);
  return used <= capacity;
}

// A run's last group is decoded when nothing is left to copy.  Where all of items[first ..] fit into one slot, returns where
// the group had better end so that a smaller one follows, whose copy hides this one's decode: before the shortest tail that
// holds an eighth of the bytes (at 57 GB/s its copy takes longer than the decode of the rest), or n_items where that gains nothing.
// A further group leaves the bus idle for 16 us, what decoding 80 MB of rows takes: cut from 128 MiB on.
int cut_last_group(const kvh_load_item* items, int first, int n_items, int l, int c, size_t capacity, int n_slots) {
  if (n_slots < 2 || n_items - first < 2 || !fits_one_group(items, first, n_items, l, c, capacity)) return n_items;
  size_t total = 0, tail = 0;
  double rows = 0;  // 16-bit bytes ahead of the tail
  for (int i = first; i < n_items; ++i) {
    total += kvh_blob_size(l, items[i].n_tokens, c, items[i].level);
    rows += 4.0 * l * c * items[i].n_tokens;
  }
  int cut = n_items;
  while (cut > first + 1 && tail * 8 < total) {
    --cut;
    tail += kvh_blob_size(l, items[cut].n_tokens, c, items[cut].level);
    rows -= 4.0 * l * c * items[cut].n_tokens;
  }
  return rows >= 128.0 * (1 << 20) ? cut : n_items;
}

// ---- the allocation-free variant: its one staging slot lives in the code object -------------------------
// Each device the library runs on holds its own copy of this array, at its own address, until the process ends.
// In host code the name is only a handle for hipGetSymbolAddress; the address kernels and copies use is the one
// that call returns, looked up once per device.
static __device__ __align__(256) uint8_t scratch[KVH_STATIC_SCRATCH_BYTES];
static_assert(KVH_STATIC_SCRATCH_BYTES % 256 == 0 && KVH_STATIC_SCRATCH_BYTES > kDescBytes + kHeaderBytes, "scratch size");

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
uint8_t* scratch_ptr[kMaxDevices];  // per device: address of `scratch` there, nullptr until first use

// Address of the current device's scratch array (nullptr on failure).
uint8_t* scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    scratch_ptr[dev] = static_cast<uint8_t*>(p);
  }
  return scratch_ptr[dev];
}

}  // namespace
}  // namespace kvh

struct kvh_loader {
  uint8_t* staging;
  size_t slot_bytes;  // capacity of a slot for blobs (the descriptor area is extra)
  size_t slot_pitch;
  int n_slots;
  int next_slot;
  hipStream_t copy_stream;
  hipEvent_t* copied;  // [slot] the slot's group has arrived
  hipEvent_t* freed;   // [slot] the decode that read the slot has finished
  hipEvent_t entered;  // the caller's stream at the start of a run
  bool* in_use;        // [slot] `freed` has been recorded at least once
};

namespace kvh {
namespace {

void destroy(kvh_loader* ld) {
  if (ld == nullptr) return;
  if (ld->copy_stream != nullptr) (void)hipStreamDestroy(ld->copy_stream);
  if (ld->entered != nullptr) (void)hipEventDestroy(ld->entered);
  for (int s = 0; s < ld->n_slots; ++s) {
    if (ld->copied != nullptr && ld->copied[s] != nullptr) (void)hipEventDestroy(ld->copied[s]);
    if (ld->freed != nullptr && ld->freed[s] != nullptr) (void)hipEventDestroy(ld->freed[s]);
  }
  delete[] ld->copied;
  delete[] ld->freed;
  delete[] ld->in_use;
  delete ld;
}

}  // namespace
}  // namespace kvh

using namespace kvh;

extern "C" {

int kvh_loader_create(kvh_loader** out, void* staging_dev, size_t staging_bytes, int n_slots) {
  if (out == nullptr) return KVH_E_ARG;
  *out = nullptr;
  if (staging_dev == nullptr || n_slots < 1 || n_slots > kMaxSlots) return KVH_E_ARG;
  if ((reinterpret_cast<uintptr_t>(staging_dev) & 15u) != 0) return KVH_E_ALIGN;
  const size_t pitch = (staging_bytes / (size_t)n_slots) & ~size_t(15);
  if (pitch < kDescBytes + (size_t)kHeaderBytes) return KVH_E_SIZE;
  kvh_loader* ld = new (std::nothrow) kvh_loader{};
  if (ld == nullptr) return KVH_E_HIP;
  ld->staging = static_cast<uint8_t*>(staging_dev);
  ld->slot_pitch = pitch;
  ld->slot_bytes = pitch - kDescBytes;
  ld->n_slots = n_slots;
  ld->copied = new (std::nothrow) hipEvent_t[n_slots]();
  ld->freed = new (std::nothrow) hipEvent_t[n_slots]();
  ld->in_use = new (std::nothrow) bool[n_slots]();
  bool ok = ld->copied != nullptr && ld->freed != nullptr && ld->in_use != nullptr;
  // default priority; non-blocking so that the legacy default stream does not serialise the copies
  ok = ok && hipStreamCreateWithFlags(&ld->copy_stream, hipStreamNonBlocking) == hipSuccess;
  ok = ok && hipEventCreateWithFlags(&ld->entered, hipEventDisableTiming) == hipSuccess;
  for (int s = 0; ok && s < n_slots; ++s) {
    ok = hipEventCreateWithFlags(&ld->copied[s], hipEventDisableTiming) == hipSuccess &&
         hipEventCreateWithFlags(&ld->freed[s], hipEventDisableTiming) == hipSuccess;
  }
  if (!ok) {
    destroy(ld);
    return KVH_E_HIP;
  }
  *out = ld;
  return KVH_OK;
}

int kvh_loader_destroy(kvh_loader* ld) {
  if (ld == nullptr) return KVH_E_ARG;
  // the copies enqueued by this loader must not outlive it: those on its stream, and those of runs of one group, which are
  // done when their slot is free (the event of a captured run cannot be waited for, and need not be: nothing has run yet)
  const bool ok = hipStreamSynchronize(ld->copy_stream) == hipSuccess;
  for (int s = 0; s < ld->n_slots; ++s)
    if (ld->in_use[s] && hipEventSynchronize(ld->freed[s]) != hipSuccess) (void)hipGetLastError();
  destroy(ld);
  return ok ? KVH_OK : KVH_E_HIP;
}

size_t kvh_loader_slot_bytes(const kvh_loader* ld) { return ld == nullptr ? 0 : ld->slot_bytes; }

int kvh_loader_run(kvh_loader* ld, const kvh_load_item* items, int n_items, kvh_dtype dt, int l, int c,
                   const kvh_kv_view* dst, int block_tokens, int32_t* status_dev, void* stream) {
  if (ld == nullptr) return KVH_E_ARG;
  if (int rc = validate_load(items, n_items, dt, l, c, dst, block_tokens, ld->slot_bytes)) return rc;
  hipStream_t compute = static_cast<hipStream_t>(stream);
  // A run that fits into one slot has no copy for a decode to hide behind and stays on the caller's stream: waits across streams
  // would cost 25 us (4 MiB copied and decoded: 115 us on two streams, 90 on one).
  const bool one_group = fits_one_group(items, 0, n_items, l, c, ld->slot_bytes);
  hipStream_t copies = one_group ? compute : ld->copy_stream;
  // Stream order: the copies read host blobs that work already enqueued on the caller's stream may
  // still be writing (an encode straight into pinned memory), so they start after that work.
  if (!one_group &&
      (hipEventRecord(ld->entered, compute) != hipSuccess || hipStreamWaitEvent(copies, ld->entered, 0) != hipSuccess))
    return KVH_E_HIP;
  DecodeParams a{};
  a.k = static_cast<uint16_t*>(dst->k);
  a.v = static_cast<uint16_t*>(dst->v);
  a.layer_stride = dst->layer_stride;
  a.token_stride = dst->token_stride;
  a.l = l;
  a.c = c;
  a.block_tokens = block_tokens;
  a.split = kNoSplit;
  int first = 0, last = n_items;  // last: where the group being packed has to end
  while (first < n_items) {
    const int s = ld->next_slot;
    uint8_t* slot = ld->staging + (size_t)s * ld->slot_pitch;
    CopyGroup g{};
    int max_tokens = 0;
    bool raw = false;
    if (!one_group && last == n_items) last = cut_last_group(items, first, n_items, l, c, ld->slot_bytes, ld->n_slots);
    pack_group(items, first, last, l, c, slot, ld->slot_bytes, g, max_tokens, raw);
    if (first + g.n == last) last = n_items;
    // the slot may still be read by the decode that used it last (in this run or an earlier one)
    if (ld->in_use[s] && hipStreamWaitEvent(copies, ld->freed[s], 0) != hipSuccess) return KVH_E_HIP;
    if (int rc = launch_copy(g, slot, copies)) return rc;
    a.kept_items = reinterpret_cast<const kvh_kept_item*>(slot);
    a.status = status_dev != nullptr ? status_dev + first : nullptr;
    int rc = KVH_OK;
    if (!one_group && (hipEventRecord(ld->copied[s], copies) != hipSuccess || hipStreamWaitEvent(compute, ld->copied[s], 0) != hipSuccess))
      rc = KVH_E_HIP;
    if (rc == KVH_OK) rc = launch_decode(a, dt, g.n, max_tokens, raw, compute);
    if (rc == KVH_OK && hipEventRecord(ld->freed[s], compute) != hipSuccess) rc = KVH_E_HIP;
    if (rc != KVH_OK) {
      // No event tells a later run, which may be on another stream, when the slot is free: both the copy that writes it and a
      // decode that may already read it are waited for here.
      (void)hipStreamSynchronize(copies);
      if (!one_group) (void)hipStreamSynchronize(compute);
      return rc;
    }
    ld->in_use[s] = true;
    ld->next_slot = (s + 1) % ld->n_slots;
    first += g.n;
  }
  return KVH_OK;
}

int kvh_load_static(const kvh_load_item* items, int n_items, kvh_dtype dt, int l, int c, const kvh_kv_view* dst,
                    int block_tokens, int32_t* status_dev, void* stream) {
  constexpr size_t capacity = (size_t)KVH_STATIC_SCRATCH_BYTES - kDescBytes;
  if (int rc = validate_load(items, n_items, dt, l, c, dst, block_tokens, capacity)) return rc;
  uint8_t* slot = scratch_on_current_device();
  if (slot == nullptr) return KVH_E_HIP;
  hipStream_t compute = static_cast<hipStream_t>(stream);
  DecodeParams a{};
  a.k = static_cast<uint16_t*>(dst->k);
  a.v = static_cast<uint16_t*>(dst->v);
  a.layer_stride = dst->layer_stride;
  a.token_stride = dst->token_stride;
  a.l = l;
  a.c = c;
  a.block_tokens = block_tokens;
  a.split = kNoSplit;
  // One slot, one stream: copy group, decode group, copy the next group over it.  Stream order keeps a copy from
  // overtaking the decode that still reads the slot; nothing in the slot has to start at zero (the copy kernel
  // rewrites the descriptors of every group).
  for (int first = 0; first < n_items;) {
    CopyGroup g{};
    int max_tokens = 0;
    bool raw = false;
    pack_group(items, first, n_items, l, c, slot, capacity, g, max_tokens, raw);
    if (int rc = launch_copy(g, slot, compute)) return rc;
    a.kept_items = reinterpret_cast<const kvh_kept_item*>(slot);
    a.status = status_dev != nullptr ? status_dev + first : nullptr;
    if (int rc = launch_decode(a, dt, g.n, max_tokens, raw, compute)) return rc;
    first += g.n;
  }
  return KVH_OK;
}

}  // extern "C"
