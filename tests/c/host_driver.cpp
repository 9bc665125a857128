// The library's host side against a stand-in for the HIP runtime, without a GPU:
// this program defines the runtime's entry points (its own symbols come before
// the shared runtime's), so libaqs.so runs on them.  Streams are queues whose
// work is done only when somebody waits for it, which makes a missing wait show
// every time; kernels are recorded by name, and those a scenario needs change
// the states as the real ones would.
//
//   host_driver SCENARIO      exit status 0 and "ok", or what was wrong
#include <algorithm>
#include <cctype>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "aqs.h"
#include "kernels.h"
#include "learned.h"
#include "linear.h"

using namespace aqs;

namespace {

struct Stream {
  std::vector<std::function<void()>> ops;
  size_t done = 0;
  bool idle() const { return done == ops.size(); }
};
struct Event {
  Stream* s = nullptr;
  size_t at = 0;   // happened once the stream has done this many operations
  bool happened() const { return s && s->done >= at; }
};

struct Runtime {
  std::map<const void*, std::string> names;
  std::map<std::string, int> launched;   // by kernel name, template arguments left out
  std::set<Stream*> streams;
  std::map<char*, size_t> pinned_size;
  Stream null_stream;
  hipError_t last = hipSuccess;
  dim3 grid, block;
  size_t shmem = 0;
  hipStream_t stream = nullptr;
  // of the scenarios
  bool fail_capture = false, fail_pinned = false, fail_uploads = false;
  int small_pending = 0, small_unread = 0;   // k_small: in flight, launched behind one in flight
  std::vector<int> small_iters;
  int lost_ops = 0;                          // operations of streams destroyed with work in them
};
Runtime& R() {
  static Runtime r;   // the library registers its kernels before main
  return r;
}

Stream* of(hipStream_t s) { return s ? reinterpret_cast<Stream*>(s) : &R().null_stream; }
Event* of(hipEvent_t e) { return reinterpret_cast<Event*>(e); }
void drain(Stream* s, size_t upto) {
  while (s->done < upto) {
    auto op = s->ops[s->done];
    op();
    ++s->done;
  }
}
void drain(Stream* s) { drain(s, s->ops.size()); }

[[noreturn]] void wrong(const char* what) {
  std::printf("wrong: %s\n", what);
  std::exit(1);
}
void expect(bool ok, const char* what) {
  if (!ok) wrong(what);
}
void call(aqs_status st, const char* what) {
  if (st != AQS_OK) {
    std::printf("%s: %s\n", what, aqs_last_error());
    std::exit(1);
  }
}

// ---- kernels ---------------------------------------------------------------

template <class T>
T arg(void** args, int i) {
  return *reinterpret_cast<T*>(args[i]);
}

// Every minimisation of a slot converges at once; a chain with predicted starts
// waits for the host before each step, another runs through.
void small_slot(const SmallArgs& sa, int r) {
  State& s = sa.it.state[r];
  while (phase_force(s.phase)) {
    if (s.step == s.n_steps) {
      s.phase = PH_DONE;
    } else {
      ++s.step;
      s.phase = predicted_start_mode(s.start_mode) ? PH_LDESC : PH_FIRE;
    }
  }
}

std::function<void()> kernel(const std::string& name, dim3 grid, void** args) {
  if (name == "k_small") {
    const SmallArgs sa = arg<SmallArgs>(args, 0);
    const int n = (int)grid.x;
    R().small_unread += R().small_pending > 0 ? 1 : 0;
    R().small_iters.push_back(sa.iters);
    ++R().small_pending;
    return [sa, n] {
      for (int i = 0; i < n; ++i) small_slot(sa, sa.slots[i]);
      --R().small_pending;
    };
  }
  if (name == "k_lextrap") {   // the start has moved every atom past any skin
    const LearnArgs a = arg<LearnArgs>(args, 0);
    return [a] {
      for (int i = 0; i < a.nsel; ++i) {
        const Geom& g = a.geom[a.sel[i]];
        for (int b = 0; b < g.nblocks; ++b) a.upart[g.block0 + b] = 1.0;
      }
    };
  }
  if (name == "k_lctl") {
    const LearnArgs a = arg<LearnArgs>(args, 0);
    return [a] {
      for (int i = 0; i < a.nsel; ++i) {
        State& s = a.state[a.sel[i]];
        if (s.phase != PH_LDESC) continue;
        s.phase = PH_LPLAIN;
        s.k += 1;
      }
    };
  }
  if (name == "k_rb_back") {
    const RebuildArgs a = arg<RebuildArgs>(args, 0);
    return [a] {
      for (int i = 0; i < a.nreps; ++i) {
        const Geom& g = a.geom[a.reps[i]];
        for (int b = 0; b < g.nblocks; ++b) a.upart[g.block0 + b] = 0.0;
      }
    };
  }
  if (name == "k_load_atoms") {
    const Geom g = arg<Geom>(args, 0);
    const auto pos = arg<const double*>(args, 1);
    const auto types = arg<const uint8_t*>(args, 2);
    const auto pos4 = arg<double4*>(args, 3);
    const auto id = arg<int32_t*>(args, 4), inv = arg<int32_t*>(args, 5);
    return [=] {
      for (int i = 0; i < g.n; ++i) {
        pos4[g.atom_off + i] = make_double4(pos[2 * i], pos[2 * i + 1], 0.0, types[i]);
        id[g.atom_off + i] = inv[g.atom_off + i] = i;
      }
    };
  }
  if (name == "k_pack_positions") {
    const Geom g = arg<Geom>(args, 0);
    const auto pos4 = arg<const double4*>(args, 1);
    const auto inv = arg<const int32_t*>(args, 2);
    const auto out = arg<double*>(args, 3);
    return [=] {
      for (int i = 0; i < g.n; ++i) {
        const double4 p = pos4[g.atom_off + inv[g.atom_off + i]];
        out[2 * i] = p.x;
        out[2 * i + 1] = p.y;
      }
    };
  }
  return [] {};
}

hipError_t launch(const void* f, dim3 grid, void** args, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  // the name within the mangled one: small letters, digits and underscores
  const std::string& full = R().names[f];
  const size_t k = full.find("k_");
  expect(k != std::string::npos, "a kernel's name");
  size_t e = k;
  while (e < full.size() && (std::islower(full[e]) || std::isdigit(full[e]) || full[e] == '_')) ++e;
  const std::string name = full.substr(k, e - k);
  ++R().launched[name];
  Stream* s = of(stream);
  auto op = kernel(name, grid, args);
  if (e0) *of(e0) = Event{s, s->ops.size() + 1};
  if (e1) *of(e1) = Event{s, s->ops.size() + 1};
  s->ops.push_back(op);
  return hipSuccess;
}

}  // namespace

// ---- the runtime's entry points ----------------------------------------------

extern "C" {

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&R()); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*,
                           void*, int*) {
  R().names[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
  R().grid = grid;
  R().block = block;
  R().shmem = shmem;
  R().stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
  *grid = R().grid;
  *block = R().block;
  *shmem = R().shmem;
  *s = R().stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s) {
  return launch(f, grid, args, s, nullptr, nullptr);
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1, int) {
  return launch(f, grid, args, s, e0, e1);
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  *a = hipFuncAttributes{};
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 160 * 1024;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorNotReady ? "not ready" : "refused by the stand-in"; }
hipError_t hipGetLastError() {
  const hipError_t e = R().last;
  R().last = hipSuccess;
  return e;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidValue; }

hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (R().fail_pinned) return R().last = hipErrorOutOfMemory;
  *p = std::malloc(n);
  R().pinned_size[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (!R().pinned_size.erase((char*)p)) wrong("freeing what was not pinned");
  std::free(p);
  return hipSuccess;
}

static bool is_pinned(const void* p) {
  auto it = R().pinned_size.upper_bound((char*)const_cast<void*>(p));
  if (it == R().pinned_size.begin()) return false;
  --it;
  return (const char*)p < it->first + it->second;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t stream) {
  Stream* s = of(stream);
  if (kind == hipMemcpyHostToDevice && R().fail_uploads) return R().last = hipErrorUnknown;
  if (kind == hipMemcpyHostToDevice && !is_pinned(src)) {   // staged before the call returns
    std::vector<char> held((const char*)src, (const char*)src + n);
    s->ops.push_back([=] { std::memcpy(dst, held.data(), n); });
    return hipSuccess;
  }
  s->ops.push_back([=] { std::memcpy(dst, src, n); });
  if (kind == hipMemcpyDeviceToHost && !is_pinned(dst)) drain(s);   // returns with the data
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t s) {
  of(s)->ops.push_back([=] { std::memset(dst, v, n); });
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  Stream* q = new Stream;
  R().streams.insert(q);
  *s = reinterpret_cast<hipStream_t>(q);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  R().lost_ops += (int)(of(s)->ops.size() - of(s)->done);
  R().streams.erase(of(s));
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  drain(of(s));
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) {
  drain(of(s));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  const Event ev = *of(e);
  of(s)->ops.push_back([ev] {
    if (ev.s) drain(ev.s, ev.at);
  });
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(new Event);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete of(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  *of(e) = Event{of(s), of(s)->ops.size()};
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  if (!of(a)->happened() || !of(b)->happened()) return R().last = hipErrorNotReady;
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  return R().fail_capture ? (R().last = hipErrorStreamCaptureUnsupported) : hipErrorNotSupported;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"

// ---- scenarios -----------------------------------------------------------------

namespace {

struct Case {
  aqs_ctx* c = nullptr;
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  std::vector<std::vector<double>> pos;
  std::vector<std::vector<uint8_t>> types;

  // 2D slots of the given sizes
  explicit Case(const std::vector<int>& n, const aqs_tuning& tn = aqs_tuning{}) {
    aqs_potential pot{};
    pot.dim = 2;
    pot.rc_factor = 2.5;
    for (int a = 0; a < 2; ++a)
      for (int b = 0; b < 2; ++b) pot.eps[a][b] = pot.sigma[a][b] = 1.0;
    aqs_fire_params fire{};
    fire.dt0 = 0.01;
    fire.max_iter = 1000;
    const int R_ = (int)n.size();
    std::vector<double> box, dg(R_, 1e-4);
    for (int r = 0; r < R_; ++r)
      for (int a = 0; a < 2; ++a) box.push_back(10.0 + std::max(0, n[r] - 100) / 100.0);
    const size_t bytes = aqs_workspace_bytes(&pot, &tn, R_, n.data(), box.data());
    ws = (char*)std::aligned_alloc(256, bytes);
    call(hipStreamCreateWithFlags(&stream, 0) == hipSuccess ? AQS_OK : AQS_EHIP, "stream");
    call(aqs_create(&pot, &fire, &tn, R_, n.data(), box.data(), dg.data(), ws, bytes, stream, &c), "create");
    for (int r = 0; r < R_; ++r) {
      pos.emplace_back();
      types.emplace_back(n[r], 0);
      for (int i = 0; i < 2 * n[r]; ++i) pos[r].push_back(0.001 * i);
    }
  }
  aqs_status load(int r) { return aqs_set_replica(c, r, types[r].data(), pos[r].data(), 0); }
  void load_all() {
    for (size_t r = 0; r < pos.size(); ++r) call(load((int)r), "set_replica");
  }
};

// Every poll of a chain waits for the block before it, also where the start's
// own work (a linear response whose probes need new lists) has read states back.
void linear_start_polls(bool profiled) {
  Case k({100});
  k.load_all();
  if (profiled) call(aqs_set_profiling(k.c, 1), "profiling");
  const int32_t rep[1] = {0}, steps[1] = {3};
  call(aqs_minimize_batch(k.c, 1, rep, AQS_START_LINEAR, steps, nullptr, nullptr), "minimize");
  expect(R().launched["k_rb_back"] == 1 + 3, "lists rebuilt at the start and before each solve");
  expect(R().launched["k_lin_begin"] == 3, "one solve per step");
  expect(R().small_unread == 0, "a block was launched behind one that nobody had read back");
  expect(R().launched["k_small"] == 1 + 3, "one launch per minimisation");
  call(aqs_destroy(k.c), "destroy");
}

// Loading and copying a slot are over when the calls return.
void slot_loads_wait() {
  Case k({100, 100});
  for (int r = 0; r < 2; ++r) {
    call(k.load(r), "set_replica");
    expect(of(k.stream)->idle(), "aqs_set_replica returned with work in its stream");
  }
  call(aqs_copy_replica(k.c, 0, 1), "copy_replica");
  expect(of(k.stream)->idle(), "aqs_copy_replica returned with work in its stream");
  std::vector<double> x(200);
  call(aqs_get_positions(k.c, 0, x.data()), "get_positions");
  expect(x == k.pos[0], "the positions as they were loaded");
  call(aqs_destroy(k.c), "destroy");
}

// A launch that fails beside work on the side stream: the lane's stream still
// waits for that work, and so does the context's end.
void side_stream_joins(bool destroy) {
  aqs_tuning tn{};
  tn.use_graph = 1;
  Case k({100, 1100}, tn);   // one workgroup, and tiles
  k.load_all();
  R().fail_capture = true;
  const int32_t rep[2] = {0, 1};
  expect(aqs_minimize_batch(k.c, 2, rep, AQS_START_PLAIN, nullptr, nullptr, nullptr) == AQS_EHIP, "capture refused");
  expect(R().launched["k_small"] == 1, "the small slot's launch");
  if (!destroy) {
    expect(hipStreamSynchronize(k.stream) == hipSuccess && R().small_pending == 0,
           "the context's stream did not wait for its side stream");
  }
  call(aqs_destroy(k.c), "destroy");
  expect(R().small_pending == 0 && R().lost_ops == 0, "destroyed with work in flight");
}

// A launch of small slots alone outlasts a minimisation, so that its lists are
// not built every few iterations and a slow slot does not make a batch of
// predicted starts wait for it twice; a live round's launches are shorter, and
// beside tiles a launch ends with their block.
void small_launch_length(int start, int32_t live, int least, int most) {
  aqs_tuning tn{};
  tn.block_iters = 8;
  Case k({100, 100, 100, 100}, tn);
  k.load_all();
  const int32_t rep[3] = {0, 1, 2}, snap[2] = {-1, 3}, steps[3] = {3, 3, 3};
  aqs_check checks[2];
  if (live < 0)
    call(aqs_minimize_batch(k.c, 3, rep, start, steps, nullptr, nullptr), "minimize");
  else
    call(aqs_run_round(k.c, 2, rep, snap, steps, start, 1e-4, live, nullptr, checks), "run_round");
  for (int n : R().small_iters) expect(n >= least && n <= most, "the length of a launch");
  call(aqs_destroy(k.c), "destroy");
}

// No pinned memory left for the staging: atoms and records still get through.
void staging_without_pinned_memory() {
  Case k({100, 100});
  R().fail_pinned = true;
  k.load_all();
  const int32_t rep[2] = {0, 1}, steps[2] = {2, 2};
  aqs_step_record rec[6];
  for (aqs_step_record& r : rec) r.status = 7;
  call(aqs_minimize_batch(k.c, 2, rep, AQS_START_PLAIN, steps, nullptr, rec), "minimize");
  expect(rec[5].status == 0, "the last record");
  std::vector<double> x(200);
  call(aqs_get_positions(k.c, 1, x.data()), "get_positions");
  expect(x == k.pos[1], "the positions as they were loaded");
  expect(hipGetLastError() == hipSuccess, "an error left behind");
  call(aqs_destroy(k.c), "destroy");
}

// A call that fails before the device has its states: later calls see the
// device's, not what the call was about to write.
void failed_writes_are_not_believed() {
  Case k({100, 100});
  k.load_all();
  const int32_t rep[1] = {0};
  const int64_t dk[1] = {5};
  int64_t got = -1;
  R().fail_uploads = true;
  expect(aqs_affine_shear(k.c, 1, rep, dk) == AQS_EHIP, "a shear that cannot be uploaded");
  expect(aqs_set_replica(k.c, 1, k.types[1].data(), k.pos[1].data(), 7) == AQS_EHIP, "a load likewise");
  R().fail_uploads = false;
  (void)hipGetLastError();
  call(aqs_get_strain_index(k.c, 0, &got), "strain_index");
  expect(got == 0, "the strain index of a shear that failed");
  call(aqs_affine_shear(k.c, 1, rep, dk), "affine_shear");
  call(aqs_get_strain_index(k.c, 0, &got), "strain_index");
  expect(got == 5, "the strain index of a shear");
  call(aqs_destroy(k.c), "destroy");
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "linear_start_polls") linear_start_polls(false);
  else if (what == "linear_start_polls_profiled") linear_start_polls(true);
  else if (what == "slot_loads_wait") slot_loads_wait();
  else if (what == "side_stream_joins") side_stream_joins(false);
  else if (what == "side_stream_joins_destroy") side_stream_joins(true);
  else if (what == "length_plain") small_launch_length(AQS_START_PLAIN, -1, 2048, 2048);
  else if (what == "length_extrapolated") small_launch_length(AQS_START_EXTRAPOLATED, -1, 2048, 2048);
  else if (what == "length_linear") small_launch_length(AQS_START_LINEAR, -1, 2048, 2048);
  else if (what == "length_round") small_launch_length(AQS_START_PLAIN, 0, 2048, 2048);
  else if (what == "length_live") small_launch_length(AQS_START_PLAIN, 1, 64, 512);
  else if (what == "staging_without_pinned_memory") staging_without_pinned_memory();
  else if (what == "failed_writes_are_not_believed") failed_writes_are_not_believed();
  else wrong("no such scenario");
  std::printf("ok\n");
  return 0;
}
