"""The sizes of a render's scratch (csrc/plan.h, compiled for the CPU): what a
pass can write has room in what the call reserved."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_11510_amd", "csrc")
SHIM = """
#include "plan.h"
extern "C" void list_plan(uint64_t most, uint64_t* out) {
  const tv::ListPlan p = tv::list_plan(most);
  out[0] = p.chunk_blocks; out[1] = p.band_size; out[2] = p.words();
}
extern "C" void queue_plan(int64_t samples, int64_t waves, int64_t* out) {
  const tv::QueuePlan p = tv::queue_plan(samples, waves);
  out[0] = p.chunk; out[1] = p.chunks; out[2] = p.records(); out[3] = p.sure();
}
extern "C" void first_grid(uint64_t most, uint32_t train_blocks, uint32_t* out) {
  const tv::FirstGrid g = tv::first_grid(tv::list_plan(most), train_blocks);
  out[0] = g.x; out[1] = g.y;
}
extern "C" int64_t queued_pass(int64_t slots, int64_t most, int64_t bytes) { return tv::queued_pass(slots, most, bytes); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "plan.so"), str(d / "shim.cpp")],
                   check=True)
    return ctypes.CDLL(str(d / "plan.so"))


def lists(plan, most):
    out = (ctypes.c_uint64 * 3)()
    plan.list_plan(ctypes.c_uint64(most), out)
    return list(out)


def dealt(ne, chunk_blocks):
    """The most entry records of ne that one of the eight lists can be dealt:
    a chunk of every round of eight, the last one perhaps cut."""
    g = 64 * chunk_blocks
    full, rest = divmod(ne, 8 * g)
    return full * g + min(rest, g)


@pytest.mark.parametrize("w,h", [(8, 8), (24, 20), (64, 64), (96, 80), (192, 120), (144, 120), (192, 192), (251, 187),
                                 (640, 360), (1024, 1024)])
def test_every_pass_fits_the_lists_of_the_largest(plan, w, h):
    """A call of several passes reserves its lists for the largest; the last
    pass may have any smaller number of samples."""
    slots = ((w + 7) // 8) * ((h + 7) // 8) * 64
    caps = {c for c in (1, 2, 3, 5, 18, 30, 48, 95, 127, 272, 511, (1 << 21) // slots, (1 << 25) // slots) if 1 <= c * slots <= 1 << 25}
    for cap in caps:
        chunk, band, words = lists(plan, slots * cap)
        assert words == 8 * band and words >= slots * cap and words <= slots * cap + 8 * 64 * chunk
        for last in {1, cap, cap - 1, cap // 2, *range(max(1, cap - 40), cap + 1)} - {0}:
            assert dealt(slots * last, chunk) <= band, (cap, last)


def test_a_shorter_passes_own_plan_does_not_fit(plan):
    """Why a call has one plan: 64 x 64 pixels, passes of 272 and 271 samples."""
    assert lists(plan, 4096 * 271)[2] > lists(plan, 4096 * 272)[2]


@pytest.mark.parametrize("slots", [64, 4096, 23040, 49152, 921600, 1 << 20, 1 << 21])
def test_passes_that_queue_light_rays_in_fixed_scratch(plan, slots):
    """Entry records, lists and 1.25 light rays a sample fit beside each other."""
    plan.queued_pass.restype = ctypes.c_int64
    room = (1 << 21) * 36  # (the array has the lists' slack and the counters besides)
    for most in (1, 2, 30, (1 << 21) // slots):
        n = slots * plan.queued_pass(ctypes.c_int64(slots), ctypes.c_int64(most), ctypes.c_int64(room))
        assert n <= slots * most and 32 * n + 4 * n + 40 * n <= room
        assert n == slots * most or 76 * (n + slots) > room


@pytest.mark.parametrize("samples", [1, 64, 4096, (1 << 20) - 1, 1 << 20, 1 << 25, 1 << 30, (1 << 32) - 1])
@pytest.mark.parametrize("blocks_per_cu", [1, 8, 64, 1 << 12, 1 << 16, (1 << 31) - 1])
def test_queue_of_any_number_of_waves(plan, samples, blocks_per_cu):
    """Records are counted in 32 bits, also for launches of very many blocks;
    the usual 8 blocks per CU leave room for 4 light rays a sample."""
    out = (ctypes.c_int64 * 4)()
    plan.queue_plan(ctypes.c_int64(samples), ctypes.c_int64(256 * blocks_per_cu * 4), out)
    chunk, chunks, records, sure = out
    assert records == chunk * chunks <= 1 << 27 and chunks > 0 and 0 <= sure <= records
    if blocks_per_cu <= 8:
        assert sure > min(1 << 26, 4 * samples) - chunk


@pytest.mark.parametrize("most", [64, 4096, 1 << 25, 1 << 31, (1 << 32) - 300000, (1 << 32) - 65536, (1 << 32) - 64])
@pytest.mark.parametrize("train_blocks", [0, 8, 4096])
def test_grid_of_the_first_kernel(plan, most, train_blocks):
    """Fewer than 2^32 threads along x, every list's blocks, rows in batches
    (which have no training paths) alone, blocks dealt by eights."""
    out = (ctypes.c_uint32 * 2)()
    plan.first_grid(ctypes.c_uint64(most), ctypes.c_uint32(train_blocks), out)
    x, y = out
    blocks = train_blocks + lists(plan, most)[2] // 64
    assert x * 64 < 1 << 32 and x % 8 == 0 and blocks <= x * y < blocks + 8 * y + 8
    assert y == 1 if most <= 1 << 31 else y <= 2
    if y == 1:
        assert x == blocks
