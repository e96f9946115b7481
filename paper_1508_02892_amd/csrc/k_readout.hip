// Read-out of one discharge's state record and profiles into a host buffer.
#include "hd_device.h"

namespace hd {
namespace {

// The parts of a read-out, in the buffer's order (Readout::off); each is
// copied where its bit of `want` is set.  The buffer is pinned host memory
// that the kernel writes over the bus: one launch and one wait bring what
// took a copy of its own per array (about 25 us each), in 8-byte words whose
// 64-lane stores fill 512 bytes.  Bound by the launch and the bus round trip
// (257 nodes, 23 KB) up to the bus itself (4,097 nodes, 300 KB).
constexpr int kThreadsR = 256;
template <class P>
__global__ __launch_bounds__(kThreadsR) void k_readout(const Disch<P>* __restrict__ dp, Readout r,
                                                       uint32_t want, uint64_t* __restrict__ out) {
  const Disch<P>& d = *dp;
  const int part = blockIdx.y;
  if (!((want >> part) & 1u)) return;
  const State* st = d.st;
  const void* src = nullptr;
  switch (part) {
    case kRoState: src = st; break;
    case kRoCnt: src = d.cnt[st->cbuf]; break;
    case kRoNi: src = d.ni; break;
    case kRoGam: src = d.gam; break;
    case kRoPhi: src = d.phi; break;
    case kRoE: src = d.E; break;
    case kRoAccCnt: src = d.acc_cnt; break;
    case kRoAccNi: src = d.acc_ni; break;
    default: src = d.eedf; break;
  }
  const Gp<uint64_t>* s = gptr(static_cast<const uint64_t*>(src));
  Gp<uint64_t>* o = gptr(out + r.off[part]);
  const uint32_t n = r.off[part + 1] - r.off[part];
  for (uint32_t i = blockIdx.x * kThreadsR + threadIdx.x; i < n; i += gridDim.x * kThreadsR) o[i] = s[i];
}

}  // namespace

// r: offsets in words; out: pinned host memory of r.off[kRoParts] words.
template <class P>
hipError_t launch_readout(const Disch<P>* d, const Readout& r, uint32_t want, uint64_t* out,
                          hipStream_t s) {
  uint32_t most = 0;
  for (int k = 0; k < kRoParts; ++k) most = r.off[k + 1] - r.off[k] > most ? r.off[k + 1] - r.off[k] : most;
  const unsigned gx = (most + 4u * kThreadsR - 1u) / (4u * kThreadsR);  // four words per thread
  hipLaunchKernelGGL(k_readout<P>, dim3(gx, kRoParts), dim3(kThreadsR), 0, s, d, r, want, out);
  return hipGetLastError();
}

template hipError_t launch_readout<float>(const Disch<float>*, const Readout&, uint32_t, uint64_t*,
                                          hipStream_t);
template hipError_t launch_readout<double>(const Disch<double>*, const Readout&, uint32_t, uint64_t*,
                                           hipStream_t);

}  // namespace hd
