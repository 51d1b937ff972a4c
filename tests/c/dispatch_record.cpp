// Launchers that write down what they are asked to launch, in place of
// dv_kernels.hip: linked with dv_api.cpp they make a library whose calls run
// without a GPU and tell which kernels a call would have used
// (tests/test_dispatch_cpu.py).  One line per launch: the kernel, its direction,
// the sequences a launch holds at most, and the fields the tests look at.
#include <stdio.h>

#include <string>

#include "../../paper_2403_01876_amd/csrc/dv_internal.h"

namespace {

std::string g_log, g_out;

hipError_t record(const char* line) {
  g_log += line;
  return hipSuccess;
}
template <typename... T>
hipError_t record(const char* format, T... values) {
  char line[256];
  snprintf(line, sizeof line, format, values...);
  return record(line);
}

const char* way(int dir) { return dir == dv::kPack ? "out" : "in"; }

}  // namespace

namespace dv {

template <int N>
hipError_t launch_dense_runs(int dir, const DenseRunArgs<N>& a, uint32_t slabs, hipStream_t) {
  return record("dense %s n=%d tiles=%u slabs=%u\n", way(dir), N, a.deal.tiles, slabs);
}
template <int N>
hipError_t launch_paged(int dir, const PagedArgs<N>& a, bool wide, uint32_t slabs, hipStream_t) {
  return record("%s %s n=%d tiles=%d slabs=%u steps=%d wide=%d\n", a.owner ? "pool" : "table",
                way(dir), N, a.tiles, slabs, a.steps, (int)wide);
}
hipError_t launch_owner_clear(const OwnerArgs&, hipStream_t) { return record("owner-clear\n"); }
hipError_t launch_owner_build(const OwnerArgs& a, hipStream_t) {
  return record("owner-build b0=%d nseq=%d\n", a.b0, a.nseq);
}
template <int N>
hipError_t launch_owner_map(const OwnerMapArgs<N>& a, hipStream_t) {
  return record("owner-map n=%d chunks=%d\n", N, a.chunks);
}
hipError_t launch_block_claims(const OwnerArgs&, bool, hipStream_t) { return record("claims\n"); }
template <int N>
hipError_t launch_rows(int dir, bool even, const RowArgs<N>& a, uint32_t slabs, hipStream_t) {
  return record("rows %s n=%d units=%d slabs=%u even=%d\n", way(dir), N, a.total, slabs, (int)even);
}
template <int N>
hipError_t launch_split_rows(int dir, const RowArgs<N>& a, uint32_t slabs, hipStream_t) {
  return record("split-rows %s n=%d units=%d slabs=%u\n", way(dir), N, a.total, slabs);
}
template <int N>
hipError_t launch_split(int dir, const SplitArgs<N>& a, uint32_t slabs, hipStream_t) {
  return record("split %s n=%d tiles=%u slabs=%u tile=%d\n", way(dir), N, a.deal.tiles, slabs,
                a.tile);
}
template <int N>
hipError_t launch_copy(const CopyArgs<N>& a, uint32_t slabs, hipStream_t) {
  return record("copy n=%d units=%d slabs=%u\n", N, a.total, slabs);
}

// name's instances for both table sizes, the last argument before the slab
// count being const Args<N>&.
#define BOTH(name, ...)                                                                        \
  template hipError_t name<kSeqPerLaunch>(__VA_ARGS__<kSeqPerLaunch>&, uint32_t, hipStream_t); \
  template hipError_t name<kSeqMany>(__VA_ARGS__<kSeqMany>&, uint32_t, hipStream_t);
BOTH(launch_dense_runs, int, const DenseRunArgs)
BOTH(launch_rows, int, bool, const RowArgs)
BOTH(launch_split_rows, int, const RowArgs)
BOTH(launch_split, int, const SplitArgs)
BOTH(launch_copy, const CopyArgs)
#undef BOTH
template hipError_t launch_paged<kSeqPerLaunch>(int, const PagedArgs<kSeqPerLaunch>&, bool, uint32_t,
                                                hipStream_t);
template hipError_t launch_paged<kSeqMany>(int, const PagedArgs<kSeqMany>&, bool, uint32_t,
                                           hipStream_t);
template hipError_t launch_owner_map<kSeqPerLaunch>(const OwnerMapArgs<kSeqPerLaunch>&,
                                                    hipStream_t);
template hipError_t launch_owner_map<kSeqMany>(const OwnerMapArgs<kSeqMany>&, hipStream_t);

int noalloc_owner_map(hipStream_t, int32_t** out) {  // an address that nothing reads
  *out = reinterpret_cast<int32_t*>(uintptr_t{1} << 45);
  return 0;
}

}  // namespace dv

// The launches since the last call of this, a line each.
extern "C" __attribute__((visibility("default"))) const char* dispatch_record_take() {
  g_out.swap(g_log);
  g_log.clear();
  return g_out.c_str();
}
