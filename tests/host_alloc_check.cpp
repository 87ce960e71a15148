// The host paths of the C entry points while no memory can be had: operator new of the whole process throws (this program's own,
// which the library's calls resolve to). An exception that left a C entry would end the process. Built and run by
// tests/test_host_alloc.py with the library's path.
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <new>

#include "audiokv.h"

static bool none_left = false;
void* operator new(std::size_t n) {
    if (!none_left)
        if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main(int argc, char** argv) {
    void* lib = argc > 1 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) { std::printf("%s\n", argc > 1 ? dlerror() : "usage: host_alloc_check libaudiokv.so"); return 2; }
    const auto workspace = reinterpret_cast<decltype(&audiokv_workspace_bytes)>(dlsym(lib, "audiokv_workspace_bytes"));
    if (!workspace) return 2;
    int bad = 0;
    for (int dim : {64, 128, 256}) {
        audiokv_params p = {};
        p.size = sizeof(p);
        p.n_q_heads = 8; p.n_kv_heads = 2; p.head_dim = dim; p.window = 32; p.pool_kernel = 7; p.floor_frac = 0.1f;
        int32_t lens[300];
        for (int equal = 0; equal < 2; ++equal) {
            for (int i = 0; i < 300; ++i) lens[i] = equal ? 3000 : 100 + 37 * i;
            size_t before = 0, now = 1;
            none_left = false;
            bad += workspace(&p, 300, lens, &before) != AUDIOKV_OK;
            none_left = true;
            bad += workspace(&p, 300, lens, &now) != AUDIOKV_OK;
            none_left = false;
            bad += before != now;
        }
    }
    if (!bad) std::printf("no entry allocates\n");
    return bad ? 1 : 0;
}
