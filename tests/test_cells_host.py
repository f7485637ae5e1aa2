"""The pool of pinned cells (csh_cells.hip) as a program on the CPU, pinned memory and
operator new replaced by ones that can be told to fail: no cell is handed out twice, a
cell comes cleared, pages are given back but for one, threads may use it together, and
memory that runs out gives a null pointer, not an exception (its callers are C entry
points) and not a lost page.
"""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1210_5246_amd", "csrc")

SRC = r"""
#include <hip/hip_runtime.h>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <set>
#include <thread>
#include <vector>

static std::atomic<int> pages{0}, no_pin{0}, no_new{0};
static hipError_t pin(void** p, size_t n, unsigned)
{
    if (no_pin) return hipErrorOutOfMemory;
    ++pages;
    *p = std::aligned_alloc(64, n);
    return hipSuccess;
}
static hipError_t unpin(void* p)
{
    --pages;
    std::free(p);
    return hipSuccess;
}
void* operator new(size_t n)
{
    if (no_new) throw std::bad_alloc();
    return std::malloc(n);
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return no_new ? nullptr : std::malloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

#define hipHostMalloc pin
#define hipHostFree unpin
#include "csh_cells.hip"

#define CHECK(c) \
    do { \
        if (!(c)) { \
            std::printf("line %d: %s\n", __LINE__, #c); \
            return 1; \
        } \
    } while (0)

int main()
{
    using csh::HostCell;
    std::vector<HostCell*> held;
    std::set<HostCell*> all;
    held.reserve(200);
    // memory runs out with the first page: null, nothing lost
    no_new = 1;
    CHECK(csh::acquire_cell() == nullptr && pages == 0);
    no_new = 0;
    no_pin = 1;
    CHECK(csh::acquire_cell() == nullptr && pages == 0);
    no_pin = 0;
    for (int k = 0; k < 130; ++k) {
        HostCell* c = csh::acquire_cell();
        CHECK(c && c->flag == 0 && c->rate == 0.0 && all.insert(c).second);
        c->flag = 1;
        c->rate = 5.0;
        held.push_back(c);
    }
    CHECK(pages == 3);
    // and later: the 62 free cells of the last page, then null
    no_new = no_pin = 1;
    int got = 0;
    HostCell* more[64];
    for (; got < 64 && (more[got] = csh::acquire_cell()); ++got) CHECK(more[got]->flag == 0);
    CHECK(got == 62);
    no_pin = 0;
    CHECK(csh::acquire_cell() == nullptr && pages == 3);
    no_new = 0;
    no_pin = 1;
    CHECK(csh::acquire_cell() == nullptr && pages == 3);
    no_pin = 0;
    for (int k = 0; k < got; ++k) csh::release_cell(more[k]);
    csh::release_cell(nullptr);
    for (HostCell* c : held) csh::release_cell(c);
    CHECK(pages == 1);
    HostCell* c = csh::acquire_cell();
    CHECK(c && c->flag == 0 && pages == 1);
    csh::release_cell(c);
    CHECK(pages == 1);

    std::atomic<int> wrong{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&, t] {
            for (int r = 0; r < 300; ++r) {
                HostCell* mine[20];
                for (int k = 0; k < 20; ++k) {
                    mine[k] = csh::acquire_cell();
                    if (!mine[k] || mine[k]->flag) ++wrong;
                    mine[k]->flag = 100 * t + k + 1;
                }
                for (int k = 0; k < 20; ++k) {
                    if (mine[k]->flag != 100 * t + k + 1) ++wrong;
                    csh::release_cell(mine[k]);
                }
            }
        });
    for (auto& t : threads) t.join();
    CHECK(wrong == 0 && pages == 1);
    std::puts("ok");
    return 0;
}
"""


def test_the_pool(tmp_path):
    src, exe = str(tmp_path / "cells.hip"), str(tmp_path / "cells")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I", CSRC, src, "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout, r.stderr)
