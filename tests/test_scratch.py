"""Growth of the device buffers that a context keeps, with allocations that
fail (on the CPU, with an allocator that counts)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "me_host.h"

static std::set<void*> live;
static int fails_in = -1;  // the allocation that fails
static int get(void** p, size_t bytes) {
    if (fails_in-- == 0) {
        *p = (void*)1;  // an allocator may leave anything
        return 2;
    }
    *p = std::malloc(bytes);
    live.insert(*p);
    return 0;
}
static int put(void* p) {
    if (!live.erase(p)) {
        std::printf("freed twice\n");
        std::exit(1);
    }
    std::free(p);
    return 0;
}

int main(int, char** argv) {
    void *a = nullptr, *b = nullptr, *c = nullptr;
    int64_t cap = 0;
    auto grow = [&](int64_t n) {
        return me_regrow(n, cap, {{&a, size_t(4 * n)}, {&b, size_t(8 * n)}, {&c, size_t(8 * n)}}, get, put);
    };
    auto sound = [&](int want) {  // no pointer to a released buffer, none lost
        int held = 0;
        for (void* p : {a, b, c}) held += p ? (int)live.count(p) : 0;
        if (held != want || (int)live.size() != want) {
            std::printf("%d of %d buffers, %d live\n", held, want, (int)live.size());
            std::exit(1);
        }
    };
    if (grow(10) != 0 || cap != 10) return 2;
    sound(3);
    const int k = std::atoi(argv[1]);
    fails_in = k;
    if (grow(1000) != 2 || cap != 0) return 3;
    sound(k);
    fails_in = -1;
    if (grow(5) != 0 || cap != 5) return 4;  // smaller than the old capacity: allocated all the same
    sound(3);
    for (void* p : {a, b, c}) put(p);
}
"""


@pytest.mark.parametrize("failing", [0, 1, 2])
def test_a_failed_allocation_leaves_no_dangling_buffer(tmp_path, failing):
    src, exe = tmp_path / "scratch.cpp", tmp_path / "scratch"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2503_21935_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(failing)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
