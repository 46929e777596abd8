/* hipMalloc that refuses allocations above KBC_TEST_MALLOC_LIMIT bytes: loaded with
 * global symbols before libkbc.so, whose calls it then takes. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdlib.h>

int hipMalloc(void** p, size_t n)
{
    static int (*real)(void**, size_t);
    const char* limit = getenv("KBC_TEST_MALLOC_LIMIT");
    if (limit && n > strtoull(limit, NULL, 10)) {
        *p = NULL;
        return 2; /* hipErrorOutOfMemory */
    }
    if (!real) real = (int (*)(void**, size_t))dlsym(dlopen("libamdhip64.so", RTLD_NOW), "hipMalloc");
    return real(p, n);
}
