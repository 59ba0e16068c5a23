// CPU check that naming a step's kernel allocates nothing: the name is asked for
// at a C entry, which no exception may leave.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../paper_1710_04751_amd/csrc/lbm_internal.hpp"

static bool refuse = false;

void* operator new(std::size_t n) {
    void* p = refuse ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
    lbm::Geom g = {};
    g.keep16 = 16;
    for (int p = 0; p < 3; ++p)
        for (int q = 7; q <= 15; q += 8)
            for (int general = 0; general < 2; ++general)
                for (int threes = 0; threes < 2; ++threes) {
                    refuse = true;
                    const char* name = lbm::step_kernel_name((lbm::Prec)p, q, general != 0, threes != 0, g);
                    refuse = false;
                    std::puts(name);
                }
    return 0;
}
