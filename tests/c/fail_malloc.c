/* hipMalloc in front of the runtime's: requests of fail_bytes fail, from the one after the first
 * fail_after of them on (fail_bytes = 0: none). */
#include <stddef.h>

size_t fail_bytes = 0;
int fail_after = 0, failed = 0;
int (*real_malloc)(void **, size_t) = 0;

int hipMalloc(void **p, size_t n)
{
    if (fail_bytes && n == fail_bytes && fail_after-- <= 0) {
        failed++;
        return 2; /* hipErrorOutOfMemory */
    }
    return real_malloc(p, n);
}
