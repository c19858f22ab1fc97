// Stands in front of the runtime's hipLaunchKernel (loaded ahead of everything that calls it) and asks for a launch that the runtime refuses
// when told to.
#include <dlfcn.h>
#include <stddef.h>

struct Dim {
    unsigned x, y, z;
};

extern "C" {
int launches_until_failure = -1; // below zero: none fails

int hipLaunchKernel(const void *kernel, Dim grid, Dim block, void **args, size_t lds, void *stream)
{
    using Launch = int (*)(const void *, Dim, Dim, void **, size_t, void *);
    static const Launch real = reinterpret_cast<Launch>(dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipLaunchKernel"));
    if (launches_until_failure == 0) return real(kernel, grid, Dim{0, 0, 0}, args, lds, stream); // hipErrorInvalidConfiguration
    if (launches_until_failure > 0) --launches_until_failure;
    return real(kernel, grid, block, args, lds, stream);
}
}
