// A stand-in for the part of the HIP runtime the library calls, for tests of its host paths without a GPU: device memory is
// host memory, kernels do nothing, and a copy is carried out as late as the stream allows (when something waits for it),
// so a source that is rewritten too early shows.  Loaded with RTLD_GLOBAL before the library, whose calls then bind here.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

namespace {
enum { SUCCESS = 0, OUT_OF_MEMORY = 2, CAPTURE_UNSUPPORTED = 900, UNKNOWN = 999 };
template <class T>
struct Plain {  // the stand-in's own memory is not counted among the library's allocations
  typedef T value_type;
  Plain() {}
  template <class U> Plain(const Plain<U>&) {}
  T* allocate(size_t n) { return (T*)malloc(n * sizeof(T)); }
  void deallocate(T* p, size_t) { free(p); }
  bool operator==(const Plain&) const { return true; }
  bool operator!=(const Plain&) const { return false; }
};
struct Copy { void* dst; const void* src; size_t n; };
typedef std::vector<char, Plain<char>> Bytes;
std::vector<Copy, Plain<Copy>> pending;
std::vector<Bytes, Plain<Bytes>> done;  // what each copy read, in order
size_t n_done = 0;
struct Event { size_t upto; };
size_t malloc_limit = ~(size_t)0, largest_malloc = 0;
int capturing = 0, event_syncs = 0, fail_event_syncs = 0, allocations = 0;
long news = 0, fail_new_at = 0;
struct Kernel { const void* stub; const char* name; };
std::vector<Kernel, Plain<Kernel>> kernels;
Bytes launches;  // the names of the kernels launched, one a line, each with the argument asked for
const char* watched = nullptr;
int watched_arg = 0;

void drain(size_t upto) {
  for (; n_done < upto; ++n_done) {
    const Copy& c = pending[n_done];
    memcpy(c.dst, c.src, c.n);
    done.emplace_back((const char*)c.src, (const char*)c.src + c.n);
  }
}
void* take(size_t n) {
  if (fail_new_at > 0 && ++news == fail_new_at) return nullptr;
  return malloc(n ? n : 1);
}
}  // namespace

void* operator new(size_t n) {
  void* p = take(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new[](size_t n) { return operator new(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete[](void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete[](void* p, size_t) noexcept { free(p); }

extern "C" {
// controls
void fake_fail_new_at(long k) { news = 0; fail_new_at = k; }  // the k-th C++ allocation from now fails; 0: none
int fake_new_failed() { return fail_new_at > 0 && news >= fail_new_at; }
void fake_malloc_limit(size_t n) { malloc_limit = n; }        // larger device allocations fail
size_t fake_largest_malloc() { const size_t n = largest_malloc; largest_malloc = 0; return n; }
void fake_capturing(int on) { capturing = on; }
void fake_fail_event_syncs(int n) { fail_event_syncs = n; }
int fake_event_syncs() { return event_syncs; }
int fake_allocations() { return allocations; }  // calls that allocate or free, device or pinned
int fake_copies_done() { return (int)done.size(); }
size_t fake_copy_size(int i) { return done[i].size(); }
const char* fake_copy_data(int i) { return done[i].data(); }
void fake_watch(const char* part, int arg) { watched = part; watched_arg = arg; }  // launches whose name holds `part` tell int argument `arg`
const char* fake_launches() {  // since the last time
  static Bytes told;
  told.swap(launches);
  told.push_back(0);
  launches.clear();
  return told.data();
}

// the runtime
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels.push_back(Kernel{stub, name});
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
struct dim3 { unsigned x, y, z; };
int __hipPushCallConfiguration(dim3, dim3, size_t, void*) { return SUCCESS; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, void** s) {
  *g = *b = dim3{1, 1, 1};
  *n = 0;
  *s = nullptr;
  return SUCCESS;
}
int hipLaunchKernel(const void* stub, dim3, dim3, void** args, size_t, void*) {
  char line[512] = "?\n";
  for (const Kernel& k : kernels)
    if (k.stub == stub) {
      if (watched && strstr(k.name, watched)) snprintf(line, sizeof line, "%s %d\n", k.name, *(const int*)args[watched_arg]);
      else snprintf(line, sizeof line, "%s\n", k.name);
    }
  launches.insert(launches.end(), line, line + strlen(line));
  return SUCCESS;
}
int hipFuncSetAttribute(const void*, int, int) { return SUCCESS; }
int hipGetDevice(int* d) { *d = 0; return SUCCESS; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return SUCCESS; }
const char* hipGetErrorString(int) { return "an error of the stand-in runtime"; }
int hipGetLastError() { return SUCCESS; }
int hipGetSymbolAddress(void** p, const void*) { static char array[1 << 24]; *p = array; return SUCCESS; }
int hipMalloc(void** p, size_t n) {
  ++allocations;
  *p = nullptr;
  if (n > largest_malloc) largest_malloc = n;
  if (n > malloc_limit) return OUT_OF_MEMORY;
  *p = malloc(n ? n : 1);
  return *p ? SUCCESS : OUT_OF_MEMORY;
}
int hipFree(void* p) { ++allocations; drain(pending.size()); free(p); return SUCCESS; }  // (waits for the device)
int hipHostMalloc(void** p, size_t n, unsigned) { ++allocations; *p = malloc(n); return *p ? SUCCESS : OUT_OF_MEMORY; }
int hipHostFree(void* p) { ++allocations; drain(pending.size()); free(p); return SUCCESS; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { pending.push_back(Copy{d, s, n}); return SUCCESS; }
int hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, void*) { return SUCCESS; }
int hipMemsetAsync(void*, int, size_t, void*) { return SUCCESS; }
int hipStreamSynchronize(void*) {
  if (capturing) return CAPTURE_UNSUPPORTED;
  drain(pending.size());
  return SUCCESS;
}
int hipStreamIsCapturing(void*, int* status) { *status = capturing; return SUCCESS; }
int hipEventCreate(void** e) { *e = calloc(1, sizeof(Event)); return SUCCESS; }
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) { free(e); return SUCCESS; }
int hipEventRecord(void* e, void*) { ((Event*)e)->upto = pending.size(); return SUCCESS; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return SUCCESS; }  // (every pair that is asked about)
int hipEventSynchronize(void* e) {
  ++event_syncs;
  if (capturing) return CAPTURE_UNSUPPORTED;
  if (fail_event_syncs > 0) { --fail_event_syncs; return UNKNOWN; }
  drain(((Event*)e)->upto);
  return SUCCESS;
}
}
