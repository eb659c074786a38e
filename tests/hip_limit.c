/* hipMalloc that fails for one size: loaded (globally) before libvf.so it stands in front of the runtime's, so
 * that a test reaches what the library does without a certain buffer. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>

static size_t limit_size;
static int limit_hits;

/* allocations of this many bytes fail from now on (0: none does); returns how many have failed so far */
int limit(size_t bytes) { limit_size = bytes; return limit_hits; }

int hipMalloc(void **p, size_t n) {
  static int (*real)(void **, size_t);
  if (!real) {
    void *h = dlopen("libamdhip64.so.7", RTLD_NOLOAD | RTLD_LAZY); /* (the one that is in the process) */
    if (h) real = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
    if (!real) return 1;
  }
  if (n && n == limit_size) {
    ++limit_hits;
    *p = NULL;
    return 2; /* hipErrorOutOfMemory */
  }
  return real(p, n);
}
