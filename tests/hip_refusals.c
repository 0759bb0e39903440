/* Stands in front of three calls of the HIP runtime (loaded with RTLD_GLOBAL before the library under test), so that a test can have
 * one of them refused from the host: hip_refuse("name of a kernel", k) refuses that kernel's launch after k more that go
 * through, hip_refuse("hipHostMalloc", k) an allocation of pinned memory.  A refused launch never reaches the GPU.  With a k that is never
 * reached nothing is refused, and the launches are counted (hip_seen, hip_seen_grid). */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
static char what[128];
static int left, seen, pending;
static unsigned grid_x;

static int find(struct dl_phdr_info *i, size_t n, void *out) {
  (void)n;
  if (!strstr(i->dlpi_name, "libamdhip64")) return 0;
  *(void **)out = dlopen(i->dlpi_name, RTLD_LAZY | RTLD_NOLOAD);
  return 1;
}
static void *runtime(const char *sym) {
  static void *lib;
  if (!lib) dl_iterate_phdr(find, &lib);
  return dlsym(lib, sym);
}
static int refuse(const char *name, int error) {
  if (!what[0] || !name || !strstr(name, what)) return 0;
  ++seen;
  if (left-- > 0) return 0;
  what[0] = 0;
  return pending = error;
}

void hip_refuse(const char *name, int after) { strncpy(what, name, sizeof what - 1); left = after; seen = 0; }
int hip_refused(void) { return what[0] == 0; }
int hip_seen(void) { return seen; }   /* such calls since hip_refuse */
unsigned hip_seen_grid(void) { return grid_x; }   /* x of the grid of the last such launch */

int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  static int (*next)(const void *, dim3, dim3, void **, size_t, void *);
  Dl_info i;
  const char *name = what[0] && dladdr(f, &i) ? i.dli_sname : NULL;
  if (name && strstr(name, what)) grid_x = grid.x;
  int e = refuse(name, 9 /* hipErrorInvalidConfiguration */);
  if (e) return e;
  if (!next) next = (int (*)(const void *, dim3, dim3, void **, size_t, void *))runtime("hipLaunchKernel");
  return next(f, grid, block, args, lds, stream);
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
  static int (*next)(void **, size_t, unsigned);
  int e = refuse("hipHostMalloc", 2 /* hipErrorOutOfMemory */);
  if (e) return e;
  if (!next) next = (int (*)(void **, size_t, unsigned))runtime("hipHostMalloc");
  return next(p, n, flags);
}
int hipGetLastError(void) {
  static int (*next)(void);
  int e = pending;
  if (!next) next = (int (*)(void))runtime("hipGetLastError");
  pending = 0;
  return e ? e : next();
}
