/* Stands in front of hipMalloc for tests of what happens without room on the
 * device: of the allocations of lo <= bytes < hi the next `left` fail with
 * hipErrorOutOfMemory (2), everything else goes to the runtime. */
#include <stddef.h>

typedef int (*malloc_fn)(void **, size_t);
static malloc_fn real;
static size_t lo, hi;
static int left, failed;

void alloc_limit_real(void *fn) { real = (malloc_fn)fn; }
void alloc_limit_arm(size_t l, size_t h, int n)
{
    lo = l;
    hi = h;
    left = n;
    failed = 0;
}
int alloc_limit_failed(void) { return failed; }

int hipMalloc(void **p, size_t n)
{
    if (left > 0 && n >= lo && n < hi) {
        --left;
        ++failed;
        *p = NULL;
        return 2;
    }
    return real(p, n);
}
