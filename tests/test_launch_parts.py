"""Rules of the host that lay out launches, checked without a device, and a batch
that needs more threads than one launch may have (2^32): kernels with several
threads per event are launched in parts there, which tile the events without
gap or overlap, each below the limit."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "me_host.h"
int main(int argc, char** argv) {
    if (argc > 4) {
        std::printf("%d 0\n", me_turn_lanes_lg(std::atoll(argv[1]), std::atoi(argv[2]), std::atoll(argv[3])));
        return 0;
    }
    me_each_launch(std::atoll(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]),
                   [&](int64_t first, unsigned blocks) { std::printf("%lld %u\n", (long long)first, blocks); });
}
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    src, exe = d / "parts.cpp", d / "parts"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2503_21935_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]

    return run


# events per block: 8, 16, 32 (gluons on the quark line 3, 2, 1; g g -> t tbar g 8), 64, and 128 of 256 threads
@pytest.mark.parametrize("per,threads", [(8, 64), (16, 64), (32, 64), (64, 64), (128, 256)])
@pytest.mark.parametrize("nevt", [0, 1, 8, 2**28 - 1, 2**28, 2**28 + 1, 2**29 - 1, 2**29, 2**29 + 1, 2**30, 2**31 - 1, 2**32 + 5])
def test_parts_tile_the_events(parts, nevt, per, threads):
    done = 0
    for first, blocks in parts(nevt, per, threads):
        assert first == done and 0 < blocks and blocks * threads < 2**32
        done = min(nevt, first + blocks * per)
    assert done == nevt


@pytest.mark.parametrize("turn", [65536, 16384, 0])
@pytest.mark.parametrize("nhel", [16, 64, 128])
@pytest.mark.parametrize("nevt", [1, 2, 255, 256, 257, 8192, 8193, 16384, 32767, 32768, 32769, 65536, 2**31 - 1])
def test_lanes_of_single_helicities(parts, nevt, nhel, turn):
    """The largest power of two that stays within one turn, 64 and the helicities."""
    ((lg, _),) = parts(nevt, nhel, turn, "lanes")
    fits = [k for k in range(7) if 1 << k <= nhel and (k == 0 or nevt << k <= turn)]
    assert lg == max(fits)


@pytest.mark.gpu
def test_more_events_than_one_launch_holds():
    """g g -> t tbar g at eight lanes per event: 2^29 + 64 events (86 GB), 64 points over and over."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_21935_amd as me
    from inputs import process_points

    torch.cuda.empty_cache()
    n = 2**29 + 64
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 100 GB of device memory")
    m = me.MatrixElement("gg_ttg")
    pts = torch.from_numpy(process_points("gg_ttg", 64, 71)).cuda()
    want = m.eval(pts)
    mom = pts.repeat(n // 64, 1, 1)
    out = torch.full((n,), -7.0, dtype=torch.float64, device="cuda")
    m.eval(mom, out)
    assert torch.equal(out.view(-1, 64).amin(0), want) and torch.equal(out.view(-1, 64).amax(0), want)
    m.close()
    del mom, out
    torch.cuda.empty_cache()
