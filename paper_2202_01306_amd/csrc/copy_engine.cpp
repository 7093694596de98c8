// Why not hipMemcpyAsync, and why not kernels that store to the host.  The device has sixteen copy engines.  The first four
// sit beside the host link and move 55 GB/s each way; the others reach 49 GB/s and less towards the device and only 7 to
// 13 GB/s towards the host (measured, 16 MiB copies).  The runtime spreads a stream's copies over whichever engines look
// free and looks again every few copies, so that a transfer of hundreds of copies sooner or later runs at a quarter of
// the link's rate.  Kernels that store to host memory reach 42 GB/s beside matrix products and slow those down by 45 to 80 %;
// a copy engine does not slow them down at all (110 against 110 us per 4096^3 product) and both directions together move
// 93 GB/s against 74.  So copies go to engines named here, one logical queue each, through the HSA runtime that HIP itself
// runs on.
//
// An engine works its copies off in order and polls the signals a copy waits for, so a logical queue needs no stream: the
// signals of kernels (k_signal) and of other queues' copies are dependencies of the copy itself.
#include "copy_engine.h"

#include <hip/hip_runtime.h>
#include <hsa/amd_hsa_signal.h>
#include <hsa/hsa.h>
#include <hsa/hsa_ext_amd.h>

#include <algorithm>
#include <cstddef>
#include <cstdlib>
#include <cstring>

namespace hmy {

namespace {

// hipMallocSignalMemory returns the address of the value inside an HSA signal
hsa_signal_t handle_of(Signal s) {
  hsa_signal_t h;
  h.handle = reinterpret_cast<uint64_t>(s) - offsetof(amd_signal_t, value);
  return h;
}

// the agent whose memory p lies in; false for memory that the HSA runtime did not allocate
bool owner_of(const void *p, uint64_t bytes, hsa_agent_t *agent, hsa_device_type_t *kind) {
  hsa_amd_pointer_info_t info;
  std::memset(&info, 0, sizeof(info));
  info.size = sizeof(info);
  if (hsa_amd_pointer_info(p, &info, nullptr, nullptr, nullptr) != HSA_STATUS_SUCCESS) return false;
  if (info.type != HSA_EXT_POINTER_TYPE_HSA) return false;
  if (static_cast<const char *>(p) + bytes > static_cast<const char *>(info.agentBaseAddress) + info.sizeInBytes) return false;
  *agent = info.agentOwner;
  return hsa_agent_get_info(*agent, HSA_AGENT_INFO_DEVICE, kind) == HSA_STATUS_SUCCESS;
}

}  // namespace

static void store_signal(Signal s, int64_t v) { hsa_signal_store_screlease(handle_of(s), v); }

struct CopyEngines::Impl {
  hsa_agent_t gpu, cpu;
  hsa_amd_sdma_engine_id_t engine[COPY_QUEUES];
  std::vector<Signal> signals;
  size_t used = 0;
  SignalWatch watch{store_signal};
  bool probing = true;   // create()'s own copies, each waited for at once, are not watched
  // for tests: the copy of that number (from 1) fails; every so many are refused
  uint64_t copies = 0, fail_at = 0, refuse_every = 0;
};

CopyEngines *CopyEngines::create(void *dev) {
  if (const char *e = std::getenv("HMY_COPY_ENGINES"))   // 0: for tests and measurements of the streams' own copies
    if (std::atoi(e) == 0) return nullptr;
  if (hsa_init() != HSA_STATUS_SUCCESS) return nullptr;   // counts the users of the instance that HIP has initialised
  CopyEngines *c = new CopyEngines;
  c->p = new Impl;
  hsa_device_type_t kind;
  void *probe = nullptr;
  bool ok = owner_of(dev, 256, &c->p->gpu, &kind) && kind == HSA_DEVICE_TYPE_GPU;
  ok = ok && hipHostMalloc(&probe, 4096, hipHostMallocDefault) == hipSuccess;
  ok = ok && owner_of(probe, 4096, &c->p->cpu, &kind) && kind == HSA_DEVICE_TYPE_CPU;
  c->p->engine[COPY_IN] = HSA_AMD_SDMA_ENGINE_1;
  c->p->engine[COPY_STATE_IN] = HSA_AMD_SDMA_ENGINE_2;
  c->p->engine[COPY_OUT] = HSA_AMD_SDMA_ENGINE_0;
  for (int q = 0; ok && q < COPY_QUEUES; ++q) {
    // one small copy on each: the engine exists and its signals are the ones expected here
    Signal s = c->take();
    volatile hsa_signal_value_t *value = nullptr;
    ok = s && hsa_amd_signal_value_pointer(handle_of(s), &value) == HSA_STATUS_SUCCESS &&
         reinterpret_cast<Signal>(const_cast<hsa_signal_value_t *>(value)) == s;
    // out first, so that what comes in again is what was there
    ok = ok && c->copy(COPY_OUT, probe, dev, 256, {}, s);
    ok = ok && c->wait(s);
    Signal t = ok ? c->take() : nullptr;
    ok = t && c->copy(CopyQueue(q), q == COPY_OUT ? probe : dev, q == COPY_OUT ? dev : probe, 256, {}, t);
    ok = ok && c->wait(t);
  }
  if (probe) hipHostFree(probe);
  (void)hipGetLastError();
  if (!ok) {
    delete c;
    return nullptr;
  }
  c->recycle();
  c->p->copies = 0;
  c->p->probing = false;
  auto from_env = [](const char *name) { return std::getenv(name) ? uint64_t(std::max(0, std::atoi(std::getenv(name)))) : 0; };
  c->p->fail_at = from_env("HMY_FAIL_COPY");
  c->p->refuse_every = from_env("HMY_REFUSE_COPIES");
  return c;
}

CopyEngines::~CopyEngines() {
  const std::vector<Signal> signals = p->signals;
  delete p;   // the thread that looks at them
  for (Signal s : signals) hipFree(s);
  hsa_shut_down();
}

bool CopyEngines::reaches(const void *ptr, uint64_t bytes) const {
  hsa_agent_t a;
  hsa_device_type_t kind;
  return owner_of(ptr, bytes, &a, &kind) && kind == HSA_DEVICE_TYPE_CPU;
}

Signal CopyEngines::take() {
  if (p->used == p->signals.size()) {
    void *s = nullptr;
    if (hipExtMallocWithFlags(&s, 8, hipMallocSignalMemory) != hipSuccess) return nullptr;
    p->signals.push_back(static_cast<Signal>(s));
  }
  Signal s = p->signals[p->used++];
  hsa_signal_store_relaxed(handle_of(s), 1);
  return s;
}

void CopyEngines::recycle() {
  p->used = 0;
  p->watch.clear();
}

bool CopyEngines::copy(CopyQueue q, void *dst, const void *src, uint64_t bytes, const std::vector<Signal> &deps, Signal done) {
  std::vector<hsa_signal_t> d;
  d.reserve(deps.size());
  for (Signal s : deps) d.push_back(handle_of(s));
  if (++p->copies == p->fail_at) {   // as an engine leaves it: nothing copied, the signal negative
    store_signal(done, -1);
    p->watch.add(done);
    return true;
  }
  if (p->refuse_every && p->copies % p->refuse_every == 0) return false;
  const hsa_agent_t from = q == COPY_OUT ? p->gpu : p->cpu, to = q == COPY_OUT ? p->cpu : p->gpu;
  if (hsa_amd_memory_async_copy_on_engine(dst, to, src, from, bytes, uint32_t(d.size()), d.empty() ? nullptr : d.data(),
                                          handle_of(done), p->engine[q], false) != HSA_STATUS_SUCCESS)
    return false;
  if (!p->probing) p->watch.add(done);
  return true;
}

void CopyEngines::set(Signal s) { store_signal(s, 0); }

bool CopyEngines::happened(Signal s) { return p->watch.over(s); }

bool CopyEngines::wait(Signal s) {
  while (!p->watch.over(s)) hsa_signal_wait_scacquire(handle_of(s), HSA_SIGNAL_CONDITION_LT, 1, UINT64_MAX, HSA_WAIT_STATE_BLOCKED);
  return p->watch.settle();
}

bool CopyEngines::failed() { return !p->watch.settle(); }

void CopyEngines::time_copies() { hsa_amd_profiling_async_copy_enable(true); }

bool CopyEngines::times(Signal s, double *begin, double *end) {
  hsa_amd_profiling_async_copy_time_t t;
  uint64_t hz = 0;
  if (hsa_amd_profiling_get_async_copy_time(handle_of(s), &t) != HSA_STATUS_SUCCESS || t.end < t.start) return false;
  if (hsa_system_get_info(HSA_SYSTEM_INFO_TIMESTAMP_FREQUENCY, &hz) != HSA_STATUS_SUCCESS || !hz) return false;
  *begin = double(t.start) / double(hz);
  *end = double(t.end) / double(hz);
  return true;
}

}  // namespace hmy
