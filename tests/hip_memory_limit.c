/* hipMalloc, hipFree and hipMemGetInfo with a budget, for tests of what the
 * library does on a full device without filling one. Loaded with its symbols
 * global before the HIP runtime, so that the library's calls come here; they go
 * on to the runtime whose path limit_open was given. */
#include <dlfcn.h>
#include <stddef.h>

#define MOST 65536
static int (*real_malloc)(void **, size_t);
static int (*real_free)(void *);
static int (*real_info)(size_t *, size_t *);
static struct { void *p; size_t bytes; } live[MOST];
static size_t budget, used, asked;
static int armed;

int limit_open(const char *runtime)
{
  void *h = dlopen(runtime, RTLD_LAZY | RTLD_NOLOAD);
  if (!h) return 1;
  real_malloc = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
  real_free = (int (*)(void *))dlsym(h, "hipFree");
  real_info = (int (*)(size_t *, size_t *))dlsym(h, "hipMemGetInfo");
  return !(real_malloc && real_free && real_info);
}

/* from here on allocations may add up to this much (limit_off: no limit) */
void limit_set(size_t bytes) { budget = bytes; used = asked = 0; armed = 1; }
void limit_off(void) { used = asked = 0; armed = 0; }
/* bytes that calls asked for and got since then */
size_t limit_asked(void) { return asked; }

int hipMalloc(void **p, size_t bytes)
{
  if (armed && used + bytes > budget) return 2; /* hipErrorOutOfMemory */
  int e = real_malloc(p, bytes);
  if (e) return e;
  asked += bytes;
  used += bytes;
  for (int i = 0; i < MOST; i++)
    if (!live[i].p) {
      live[i].p = *p;
      live[i].bytes = bytes;
      break;
    }
  return 0;
}

int hipFree(void *p)
{
  for (int i = 0; p && i < MOST; i++)
    if (live[i].p == p) {
      used = used > live[i].bytes ? used - live[i].bytes : 0;
      live[i].p = 0;
      break;
    }
  return real_free(p);
}

int hipMemGetInfo(size_t *f, size_t *t)
{
  int e = real_info(f, t);
  if (!e && armed && *f > budget - used) *f = budget - used;
  return e;
}
