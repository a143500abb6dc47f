"""How the live pass cuts and orders its work, from the library's own code
compiled for the host by itself (CPU only)."""
import ctypes
import os
import subprocess

import pytest

from tests.conftest import ROOT

SOURCE = """
#include "cdt_device.hpp"
#include "cdt_launch.hpp"
#include <vector>
extern "C" uint64_t eighths(uint64_t it, uint64_t total, uint64_t per_shard) {
    return cdt::shard_eighths(it, total, per_shard);
}
// Workgroups of `runs` runs over one reference of `blocks` blocks of n8 groups.
extern "C" uint64_t plan(uint32_t runs, uint32_t blocks, uint32_t n8, uint32_t* per_unit) {
    const uint64_t all = static_cast<uint64_t>(runs) * blocks * n8;
    std::vector<cdt::BatchKey> keys(runs, cdt::BatchKey{nullptr, 0, 1, blocks, n8, 0, 0});
    std::vector<cdt::BatchGroupDev> groups(runs);
    uint32_t n = 0;
    cdt::group_batch_jobs(runs, keys.data(), cdt::sim_unit_runs(all), groups.data(), &n);
    if (n != 1) return 0;
    const cdt::GenShape g = cdt::gen_shape(n8, all, groups[0].jobs_per_iter);
    if (g.cpb * g.chunk_groups < n8 || (g.cpb - 1) * g.chunk_groups >= n8) return 0;
    groups[0].chunks = g.cpb * blocks;
    *per_unit = groups[0].jobs_per_iter;
    const uint64_t padded = cdt::place_batch_groups(groups.data(), n);
    const uint64_t wgs = groups[0].chunks * groups[0].units;
    return padded >= wgs && padded < wgs + 8 * groups[0].units ? wgs : 0;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.hip").write_text(SOURCE)
    so = str(d / "plan.so")
    subprocess.run([hipcc, "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "paper_2607_19490_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), str(d / "plan.hip"), "-o", so],
                   check=True, capture_output=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def plan(host):
    fn = host.plan
    fn.argtypes = [ctypes.c_uint32] * 3 + [ctypes.POINTER(ctypes.c_uint32)]
    fn.restype = ctypes.c_uint64

    def call(runs, blocks, n8):
        per = ctypes.c_uint32()
        return fn(runs, blocks, n8, ctypes.byref(per)), per.value
    return call


@pytest.mark.parametrize("blocks,n8", [(32, 512), (128, 1024), (256, 2048), (360, 4608),
                                       (1200, 4608), (512, 32768), (1024, 131072), (6, 1),
                                       (4096, 257), (3, 100003), (1000, 255)])
def test_joint_runs_leave_the_chip_full(plan, blocks, n8):
    """Runs are put together, and chunks made longer, only while 1024
    workgroups remain, or as many as one run and one group per thread give
    where that is fewer."""
    seen = set()
    for runs in (1, 2, 3, 4, 5, 6, 9, 24):
        wgs, per_unit = plan(runs, blocks, n8)
        alone = -(-n8 // 256) * blocks * runs
        assert 1 <= per_unit <= min(runs, 4)
        assert min(1024, alone) <= wgs <= alone, (runs, wgs, per_unit)
        seen.add(per_unit)
    if blocks * n8 >= 1 << 20:  # large enough for units of every size
        assert seen == {1, 2, 3, 4}


@pytest.mark.parametrize("shards", [1, 2, 16, 17])
@pytest.mark.parametrize("per_shard", [1, 7, 8, 9, 24, 61, 64])
def test_shard_eighths(host, shards, per_shard):
    """Every chunk once; an XCD's chunks of a shard follow one another."""
    fn = host.eighths
    fn.argtypes, fn.restype = [ctypes.c_uint64] * 3, ctypes.c_uint64
    total = shards * per_shard
    order = [fn(it, total, per_shard) for it in range(total)]
    assert sorted(order) == list(range(total))
    eighth = per_shard // 8
    for x in range(8):
        mine = order[x:shards * eighth * 8:8]
        assert mine == [s * per_shard + x * eighth + i for s in range(shards)
                        for i in range(eighth)]
