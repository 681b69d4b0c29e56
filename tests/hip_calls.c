/* HIP runtime calls of the library under test, counted and made to fail.
 * Loaded with RTLD_GLOBAL before the library, it stands in front of a few HIP
 * functions and passes every call on to the loaded runtime, except those that
 * the test told it to refuse. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

enum { kOk = 0, kOutOfMemory = 2, kUnknown = 999 };

static char log_[4096];
static size_t used_;
static int logging_, refuse_pinned_, sync_left_ = -1;

/* 'E' an event recorded, 'L' a kernel launched, since calls_start() */
void calls_start(void) { used_ = 0; logging_ = 1; memset(log_, 0, sizeof(log_)); }
const char* calls_end(void) { logging_ = 0; return log_; }
/* pinned host memory is refused while on is nonzero */
void calls_refuse_pinned(int on) { refuse_pinned_ = on; }
/* the left-th following synchronisation waits, then reports an error (0: the
 * next one); negative: none does */
void calls_fail_sync(int left) { sync_left_ = left; }

static void note(char c) {
  if (logging_ && used_ + 1 < sizeof(log_)) log_[used_++] = c;
}

static int find(struct dl_phdr_info* info, size_t size, void* out) {
  (void)size;
  if (!strstr(info->dlpi_name, "libamdhip64")) return 0;
  *(void**)out = dlopen(info->dlpi_name, RTLD_NOLOAD | RTLD_LAZY);
  return 1;
}

static void* real(const char* name) {
  static void* lib;
  if (!lib) dl_iterate_phdr(find, &lib);
  return dlsym(lib, name);
}

int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
  if (refuse_pinned_) return kOutOfMemory;
  return ((int (*)(void**, size_t, unsigned))real("hipHostMalloc"))(p, bytes, flags);
}

int hipStreamSynchronize(void* stream) {
  const int st = ((int (*)(void*))real("hipStreamSynchronize"))(stream);
  if (sync_left_ < 0) return st;
  return sync_left_-- == 0 ? kUnknown : st;
}

int hipEventRecord(void* event, void* stream) {
  note('E');
  return ((int (*)(void*, void*))real("hipEventRecord"))(event, stream);
}

int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds,
                    void* stream) {
  note('L');
  return ((int (*)(const void*, dim3_t, dim3_t, void**, size_t, void*))real("hipLaunchKernel"))(
      f, grid, block, args, lds, stream);
}
