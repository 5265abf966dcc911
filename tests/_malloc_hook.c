/* Counts the calls of hipMalloc while armed, and lets one of them fail.  Loaded with global symbols before the libraries
 * that call it; the calls go on to the runtime that is loaded then. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <string.h>

int hook_armed, hook_count, hook_fail_at = -1;

int hipMalloc(void **p, size_t bytes) {
    static int (*real)(void **, size_t);
    if (!real) {
        char line[4096];
        FILE *f = fopen("/proc/self/maps", "r");
        while (f && !real && fgets(line, sizeof line, f)) {
            char *path = strchr(line, '/');
            if (!path || !strstr(path, "libamdhip64")) continue;
            path[strcspn(path, "\n")] = 0;
            void *h = dlopen(path, RTLD_LAZY | RTLD_NOLOAD);
            if (h) real = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
        }
        if (f) fclose(f);
        if (!real) return 3;
    }
    if (hook_armed && hook_count++ == hook_fail_at) { *p = NULL; return 2; }
    return real(p, bytes);
}
