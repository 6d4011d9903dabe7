// Per-device runtime state and helpers shared by the forward and backward
// drivers (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <chrono>
#include <mutex>
#include <string>
#include <vector>

#include "cqsa.h"
#include "errors.hpp"
#include "plan.hpp"

namespace cqsa {

// Waves the GPU holds at once at the inner kernels' occupancy (256 CUs x 4
// SIMDs x 2 waves), and the launch length, in rounds of them, from which the
// drivers run consecutive inner launches one after the other on the caller's
// stream: such a launch has a negligible tail, and two of them in flight only
// share the GPU (which costs time: in the backward, dQ beside dK/dV was 2-8 %
// slower than the two in turn from 8 rounds up).  Shorter launches go to two
// streams, so that one fills the other's tail.
constexpr int64_t kResidentWaves = 256 * 8;
constexpr int64_t kSerialRounds = 8;
inline bool serial_launch(int64_t waves) { return waves >= kSerialRounds * kResidentWaves; }

// Cache of small plan images on one device: kImageSlots slots of
// kImageSlotBytes for each kind of call (ordinary, no-allocation), in a fixed
// device array (2 MB, like the no-allocation scratch).  A call whose plan's
// image is here uploads nothing: the copy and the gap behind it are about 10
// us of every call, a fifth of the shortest (f32 L = 1024, H = 1, d = 64: 48.2
// -> 39.5 us).  Only calls of its kind fill and read a slot, and those run one
// after another on the device, so a slot needs no order of its own and a call
// never waits for one of the other kind.  Slots are named by the plan's serial
// number, so a new plan at an old one's address never finds its image.  Images
// above the slot size are uploaded by every call (calls that large run for
// milliseconds), as are those of calls under stream capture (a replay may
// follow any other call) and of calls whose workspace is the caller's.
constexpr int kImageSlots = 16;
constexpr size_t kImageSlotBytes = 64 << 10;
struct ImageSlot {
  uint64_t serial = 0;  // the plan whose image the slot holds (0: none)
  uint64_t used = 0;    // clock of the last call that used it
  char* at = nullptr;   // its device address
};

// The end of the last call of one kind (ordinary calls, which share the
// workspace, or no-allocation calls, which share the scratch array): the next
// call's device work runs after it.  A call under stream capture is recorded
// and not run, so it neither waits for nor records `done`: an event last
// recorded in an open capture pulls every stream that waits for it into that
// capture, and stands for no work of its own afterwards.  Calls recorded into
// one capture follow one another through `recorded`.
struct CallOrder {
  hipEvent_t done = nullptr;       // end of the last call made outside capture
  bool valid = false;
  hipEvent_t recorded = nullptr;   // end of the last call made under capture
  unsigned long long capture = 0;  // that capture's id
};
// The id of the capture that stream s records, 0 when it records none.
unsigned long long capture_id(hipStream_t s);
// At the start and the end of a call's device work on stream s, which records
// capture `cap` (0: none).
cqsa_status order_begin(const CallOrder& o, hipStream_t s, unsigned long long cap);
cqsa_status order_end(CallOrder& o, hipStream_t s, unsigned long long cap);
// Whether the device is done with the last call of the kind.
bool calls_done(const CallOrder& o);

// Pinned host buffers that the plan images of one kind of call are uploaded
// from (upload_image).
struct ImageRing {
  void* pin[2] = {nullptr, nullptr};
  size_t bytes[2] = {0, 0};
  hipEvent_t done[2] = {nullptr, nullptr};
  bool valid[2] = {false, false};
  int next = 0;
};

// Library-owned streams and caches of one device.  All streams use the
// default priority.
struct DevCtx {
  int device = -1;
  bool ready = false;
  hipStream_t copy = nullptr;   // staging copies (H2D or D2D)
  hipStream_t aux = nullptr;    // forward merges, or statistics device -> host
  hipStream_t lane = nullptr;   // second compute stream (short launches: odd forward groups, backward dQ)
  CallOrder calls[2];           // of ordinary calls [0] and no-allocation calls [1]
  void* ws = nullptr;           // cached device workspace (built-in allocator)
  size_t ws_bytes = 0;
  void* pin = nullptr;          // cached pinned host staging for host accumulation
  size_t pin_bytes = 0;
  ImageRing img_ring[2];  // of ordinary calls [0] and no-allocation calls [1]
  ImageSlot img_slot[2][kImageSlots];  // of ordinary calls [0] and no-allocation calls [1]
  uint64_t img_clock = 0;
  std::vector<hipEvent_t> sync_events;  // reusable non-timing events
  // the fixed scratch array of cqsa_forward_noalloc on this device (its device
  // address, from hipGetSymbolAddress at set-up)
  void* scratch = nullptr;
  // the inner forward's tile-decision counters (cqsa_set_tile_counting),
  // allocated on first use; calls reach them in workspace order
  unsigned long long* tile_count = nullptr;
  std::mutex mu;
};

// Non-timing events created with the context, so that a call that must not
// allocate finds its synchronisation events in place.
constexpr size_t kSetupEvents = 16;

DevCtx* device_ctx(cqsa_status* st);  // context of the current device (created on first use)

// Workspace of one call: from the caller allocator when one is installed,
// else the cached per-device buffer.
struct Workspace {
  void* ptr = nullptr;
  size_t bytes = 0;
  bool from_hook = false;
};
cqsa_status acquire_workspace(DevCtx* c, size_t bytes, Workspace* ws);
void release_workspace(DevCtx* c, Workspace* ws, hipStream_t s);
cqsa_status acquire_pinned(DevCtx* c, size_t bytes, void** out);
// Enqueues the upload of a plan image on stream s.  The bytes go through a
// ring of two pinned host buffers: a copy from pageable memory would block
// the host until the stream reached it (serialising consecutive calls), and
// an asynchronous copy must not read a plan the caller may destroy as soon
// as the call returns.  A buffer is refilled once its previous upload is done.
// by_kernel (images that go to a slot of the image cache): a small kernel reads
// the buffer; else the image is copied, that of a no-allocation call from the
// plan's own memory (its ring, made at set-up, holds one slot each).  The kernel
// is for calls that find the last one done (calls_done): a copy there, and the
// gap behind it, takes 4 to 11 us more of a new plan's first call (new tensors
// too: bf16 L = 3000 no-allocation 113.9 and 108.3 us, fp16 L = 2048 forward and
// backward 209.5 and 198.7).  Behind a call that still runs the copy is the
// shorter one (a loop over 20 plans of L = 300, H = 1, us a call: no-allocation
// 33.2 and 40.1, ordinary 36.2 and 40.2).
cqsa_status upload_image(DevCtx* c, const std::vector<uint8_t>& image, void* dst, bool by_kernel,
                         bool noalloc, hipStream_t s);

// The slot of plan p's image for a call whose stream already waits for the last
// call of its kind, or null when the call uploads the image to its workspace.
// hit: the slot holds the image.  Else it is p's to fill, in order after that
// wait.
ImageSlot* image_slot(DevCtx* c, const cqsa_plan_s* p, bool noalloc, unsigned long long cap, bool* hit);
// At the end of a call, after order_end: later calls may use the image.  A call
// that fails before that leaves the slot empty.
inline void image_done(ImageSlot* slot, const cqsa_plan_s* p) {
  if (slot) slot->serial = p->serial;
}

// Event pairs for the optional per-stage timing of the last call.
enum Stage { kStStage = 0, kStInner, kStMerge, kStFinal, kStD2H, kStCount };
struct CallRecord {
  bool timing = false;
  // tile counting of the last call: the counters' copy in pinned host memory
  // (allocated on first use, per thread) and the event after that copy
  int counted = 0;                          // counters copied (0: none)
  unsigned long long* tile_host = nullptr;
  hipEvent_t tile_done = nullptr;
  std::vector<hipEvent_t> owned;                       // destroyed on reset
  std::vector<std::pair<hipEvent_t, hipEvent_t>> spans[kStCount];
  hipEvent_t wall0 = nullptr, wall1 = nullptr;
  double host_merge_ms = 0.0;
  double host_final_ms = 0.0;
  cqsa_run_stats stats{};
  void reset();
  hipEvent_t make();                                    // timing event owned by the record
};
CallRecord& call_record();
bool timing_enabled();
bool tile_counting_enabled();
// The device's first n tile counters (n <= 8), zeroed on stream s (allocated
// on first use).
cqsa_status tile_counters_begin(DevCtx* c, hipStream_t s, int n, unsigned long long** out);
// Copies the first n counters to the call record after the work on s (the
// call's end); cqsa_last_stats reads them: [0..2] the forward's or the dQ
// kernel's decisions, [3..5] the dK/dV kernel's.
cqsa_status tile_counters_end(DevCtx* c, CallRecord& rec, hipStream_t s, int n);

// Checks shared by forward and backward.
cqsa_status check_tensor(const cqsa_tensor* t, const char* name, const cqsa_plan_t* p,
                         cqsa_dtype want, cqsa_mem where);

inline cqsa_status hip_fail(hipError_t e, const char* what) {
  return fail(CQSA_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define CQSA_HIP(expr)                                                   \
  do {                                                                   \
    hipError_t e_ = (expr);                                              \
    if (e_ != hipSuccess) {                                              \
      if (e_ == hipErrorOutOfMemory) return fail(CQSA_ERR_DEVICE_OOM, #expr); \
      return hip_fail(e_, #expr);                                        \
    }                                                                    \
  } while (0)

}  // namespace cqsa
