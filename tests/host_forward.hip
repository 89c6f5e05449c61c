// The host side of the library with every launch replaced by a note of the workspace it was given, so that a test can follow
// what a forward would have run, and on which memory, without a GPU.
#include <hip/hip_runtime.h>

#include <cstring>
#include <vector>

#define hipGetDevice(dev) (*(dev) = 0, hipSuccess)
#define hipDeviceGetAttribute(value, attribute, dev) (*(value) = 256, hipSuccess)
#include "moe_api.hip"

enum { NOTE_INDEX = 1, NOTE_SCHEDULE, NOTE_RESET, NOTE_LAYER0, NOTE_LAYER1, NOTE_DECODE0, NOTE_DECODE1 };
struct Note {
  // heads, items: addresses; stride: bytes; stream: rows of an expert up to which its weights are loaded with the non-temporal hint, or (small batches) whether they are
  int64_t kind, heads, stride, items0, items1, own_index, stream;
};
static std::vector<Note> notes;

namespace moe {
static void note(int kind, const Workspace& ws) {
  notes.push_back({kind, (int64_t)ws.queue_heads, ws.head_stride * 4, (int64_t)ws.items0, (int64_t)ws.items1, 0, 0});
}
static void note(int kind, const GemmParams& p) {
  notes.push_back({kind, (int64_t)p.queue_heads, p.head_stride * 4, (int64_t)p.items, 0, 0, p.stream_rows});
}
hipError_t launch_route_topk(const float*, int, int, int, int32_t*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_index_build(const IndexParams& p, bool schedule, hipStream_t) {
  note(NOTE_INDEX, p.ws);
  if (schedule) note(NOTE_SCHEDULE, p.ws);
  return hipSuccess;
}
hipError_t launch_index_schedule(const IndexParams& p, hipStream_t) {
  note(NOTE_SCHEDULE, p.ws);
  return hipSuccess;
}
hipError_t launch_reset_counters(const Workspace& ws, int, int, bool, hipStream_t) {
  note(NOTE_RESET, ws);
  return hipSuccess;
}
hipError_t launch_layer0(const GemmParams& p, int, int, hipStream_t) {
  note(NOTE_LAYER0, p);
  return hipSuccess;
}
hipError_t launch_layer1(const GemmParams& p, int, hipStream_t) {
  note(NOTE_LAYER1, p);
  return hipSuccess;
}
hipError_t launch_fused_layers(const GemmParams& p0, const GemmParams& p1, const FuseParams&, int, int, hipStream_t) {
  note(NOTE_LAYER0, p0);
  note(NOTE_LAYER1, p1);
  return hipSuccess;
}
hipError_t launch_decode_gemm(const DecodeParams& p, const IndexParams&, int layer1, int, int, hipStream_t) {
  notes.push_back({layer1 ? NOTE_DECODE1 : NOTE_DECODE0, 0, 0, 0, 0, p.own_index, p.b_stream});
  return hipSuccess;
}
hipError_t launch_combine(const CombineParams&, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_u32(uint32_t*, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_weights(const void*, void*, int, int, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_arrival_producer(const void*, void*, const ArrivalParams&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_tile_heights(const int32_t*, int32_t*, int, hipStream_t) { return hipSuccess; }
}  // namespace moe

// Copies out the launches noted since the last call, at most capacity of them; returns how many there were.
extern "C" int host_forward_notes(int64_t* out, int capacity) {
  const int n = (int)notes.size();
  for (int i = 0; i < n && i < capacity; i++) memcpy(out + i * (sizeof(Note) / 8), &notes[i], sizeof(Note));
  notes.clear();
  return n;
}
