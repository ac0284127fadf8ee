/* Test shim: a hipMalloc that fails for sizes in [fail_lo, fail_hi]; loaded before the
 * library, whose calls it then receives. */
#include <dlfcn.h>
#include <stddef.h>

size_t fail_lo = 1, fail_hi = 0;
int failed = 0;

int hipMalloc(void** p, size_t n) {
  static int (*real)(void**, size_t) = 0;
  if (n >= fail_lo && n <= fail_hi) {
    ++failed;
    return 2; /* hipErrorOutOfMemory */
  }
  if (!real) {
    void* hip = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    if (!hip) hip = dlopen("libamdhip64.so", RTLD_LAZY);
    real = (int (*)(void**, size_t))dlsym(hip, "hipMalloc");
  }
  return real(p, n);
}
