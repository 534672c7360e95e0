// Host-only stand-ins for the device side of the library, so that the C-ABI
// host code (map construction, argument validation, planning, workspace
// sizing) can be built by a plain C++ compiler with AddressSanitizer and
// UndefinedBehaviorSanitizer.  A launch reports an error: the sanitizer
// driver only exercises paths that stop before any launch, and an
// unexpected MLKV_ERR_HIP would show that one was reached.  Prefill launches
// succeed while stub_prefills counts them (not negative): the largest grid
// of theirs, in threads along x as the device counts them, is kept, and the
// last one's form.  Launches of decode steps succeed while stub_steps counts
// them: the last one of a whole step is kept.
#include "kernels.h"

long stub_prefills = -1, stub_prefill_threads = 0;
int stub_prefill_form = -1;
long stub_steps = -1;
mlkv::StepParams stub_step;

namespace mlkv {

namespace {
hipError_t no_device() { return hipErrorInvalidDevice; }
}  // namespace

hipError_t launch_pack(const PackParams&, hipStream_t) { return no_device(); }
hipError_t launch_layer_in(const LayerInParams&, hipStream_t) { return no_device(); }
hipError_t launch_layer_out(const LayerOutParams&, hipStream_t) { return no_device(); }
hipError_t launch_norm2(const NormParams&, hipStream_t) { return no_device(); }
hipError_t launch_qkv_epilogue(const QkvEpilogueParams&, hipStream_t) { return no_device(); }
hipError_t launch_gelu(const GeluParams&, hipStream_t) { return no_device(); }
hipError_t launch_residual(const ResidualParams&, hipStream_t) { return no_device(); }
hipError_t launch_append(const AppendParams&, int, int, hipStream_t) {
  return stub_steps < 0 ? no_device() : hipSuccess;
}
hipError_t launch_rope_table(const RopeTableParams&, hipStream_t) { return no_device(); }
hipError_t launch_cache_rows(const CacheRowsParams&, int, hipStream_t) { return no_device(); }
hipError_t launch_append_rows(const AppendRowsParams&, int, int, hipStream_t) {
  return stub_prefills < 0 ? no_device() : hipSuccess;
}
hipError_t launch_prefill(const PrefillParams& p, int head_dim, hipStream_t, hipEvent_t, hipEvent_t) {
  if (stub_prefills < 0) return no_device();
  ++stub_prefills;
  stub_prefill_form = static_cast<int>(prefill_form(p, head_dim, compute_units()));
  const long threads = static_cast<long>(p.B) * p.n_groups * 256;
  stub_prefill_threads = threads > stub_prefill_threads ? threads : stub_prefill_threads;
  return hipSuccess;
}
hipError_t launch_attention_main(const AttnParams&, int, hipStream_t, hipEvent_t, hipEvent_t,
                                 const SideProduct*) {
  return stub_steps < 0 ? no_device() : hipSuccess;
}
hipError_t launch_attention_merge(const AttnParams&, int, hipStream_t, hipEvent_t) {
  return stub_steps < 0 ? no_device() : hipSuccess;
}
hipError_t launch_step(const StepParams& p, int, hipStream_t, hipEvent_t, hipEvent_t) {
  if (stub_steps < 0) return no_device();
  ++stub_steps;
  stub_step = p;
  return hipSuccess;
}
hipError_t launch_fill(uint32_t*, size_t, uint32_t, hipStream_t) { return no_device(); }
hipError_t launch_empty_timed(int, int, hipStream_t, hipEvent_t, hipEvent_t) { return no_device(); }
hipError_t launch_stream_read_timed(const void*, size_t, uint32_t*, int, hipStream_t, hipEvent_t,
                                    hipEvent_t) {
  return no_device();
}
hipError_t scratch_for_current_device(hipStream_t, void** ptr) {
  *ptr = nullptr;
  return no_device();
}
// The planner's device facts, fixed at MI355X's: 256 compute units, three
// four-wave attention workgroups resident per compute unit.
int max_batch() { return 2048; }
int stage_floats() { return 8192; }
int resident_workgroups(int) { return 768; }
int wide_waves() { return 8; }
int compute_units() { return 256; }
int default_waves() { return 4; }

}  // namespace mlkv
