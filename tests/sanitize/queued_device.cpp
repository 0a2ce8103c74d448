// A device that only queues, for CPU tests of the host code that feeds it: the HIP runtime calls and kernel launches that capi.cpp
// makes, with every launch left in a queue until the host waits for an event behind it.  A launch remembers the pinned words that its
// kernel would read and a checksum of them; when it is carried out they have to be what they were at the launch, otherwise the host has
// overwritten or freed a buffer that the device had not read yet.  Nothing is computed.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <deque>
#include <map>
#include <vector>

#include "kernels.hpp"

namespace {

struct Read {
  const uint8_t* at;
  int64_t bytes;
  uint64_t sum;
};
struct Command {
  std::vector<Read> reads;
  hipEvent_t done;
};
std::deque<Command> queue;
std::map<const uint8_t*, size_t> pinned;       // what hipHostMalloc gave out
int64_t overwritten, launches, records, waits, since_record, most_since_record;
bool blind;                                    // the planted mistake: a wait that returns at once
uint8_t scratch[256];

uint64_t checksum(const uint8_t* p, int64_t n) {
  uint64_t h = 1469598103934665603ull;
  for (int64_t i = 0; i < n; ++i) h = (h ^ p[i]) * 1099511628211ull;
  return h;
}
bool is_pinned(const uint8_t* p, int64_t n) {
  auto it = pinned.upper_bound(p);
  if (it == pinned.begin()) return false;
  --it;
  return p + n <= it->first + it->second;
}
void carry_out_one() {
  for (const Read& r : queue.front().reads) overwritten += !is_pinned(r.at, r.bytes) || checksum(r.at, r.bytes) != r.sum;
  queue.pop_front();
}
void add(Command& c, const void* p, int64_t bytes) {
  if (bytes > 0 && is_pinned((const uint8_t*)p, bytes)) c.reads.push_back({(const uint8_t*)p, bytes, checksum((const uint8_t*)p, bytes)});
}
hipError_t launch(Command c) {
  ++launches;
  most_since_record = std::max(most_since_record, ++since_record);
  queue.push_back(std::move(c));
  return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "queued device"; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)malloc(1), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0, hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(n, 1);
  pinned[(const uint8_t*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  pinned.erase((const uint8_t*)p);
  return free(p), hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  ++records;
  since_record = 0;
  queue.push_back({{}, e});
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  ++waits;
  size_t n = queue.size();
  while (n > 0 && queue[n - 1].done != e) --n;
  if (!blind)
    while (n-- > 0) carry_out_one();
  return hipSuccess;
}

void queued_be_blind(int on) { blind = on != 0; }
// carries out what is left; [reads whose words had changed, launches, event records, waits, most launches without a record between them]
void queued_finish(int64_t* out) {
  while (!queue.empty()) carry_out_one();
  const int64_t v[] = {overwritten, launches, records, waits, most_since_record};
  for (int i = 0; i < 5; ++i) out[i] = v[i];
}
}

namespace symkv {
hipError_t static_scratch_address(int, uint8_t** p) { return *p = scratch, hipSuccess; }
hipError_t launch_attn(const DecodeArgs&, const PrefillArgs&, int, int, hipStream_t, hipEvent_t, hipEvent_t) { return launch({}); }
hipError_t launch_merge(const MergeArgs&, int, int, hipStream_t) { return launch({}); }
hipError_t launch_prologue(PrologueArgs a, hipStream_t) {
  Command c{{}, a.done};
  if (a.n_runs < 1 || a.n_runs > kPrologueRuns) add(c, a.slots, (int64_t)a.n_tokens * 4);
  add(c, a.cow, (int64_t)a.n_cow * 12);
  add(c, a.host_words, a.copy_words * 4);
  return launch(c);
}
hipError_t launch_gather(const GatherArgs& a, void*, void*, hipStream_t) {
  Command c{{}, nullptr};
  add(c, a.slots, (int64_t)a.n_tokens * 4);
  return launch(c);
}
hipError_t launch_move(const MoveArgs& a, hipStream_t) {
  Command c{{}, a.done};
  for (int32_t i = 0; i < a.n_pages && !a.near; ++i) add(c, a.src + i * 16, (a.dst[i] % 16 + 1) * 4);
  if (!a.near) add(c, a.dst, (int64_t)a.n_pages * 4);
  return launch(c);
}
hipError_t launch_swap(const SwapArgs& a, hipStream_t) {
  Command c{{}, nullptr};
  add(c, a.list, (int64_t)a.n_pages * 16);
  return launch(c);
}
hipError_t launch_calib_read(const void*, int64_t, void*, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_calib_copy(void*, const void*, int64_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_calib_mfma(float*, int, int, hipStream_t) { return hipErrorNotSupported; }
}  // namespace symkv
