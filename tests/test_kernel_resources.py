"""Resources the compiler must give some kernels for them to run as they are
written: what a source line alone does not show (CPU only)."""
import pytest

from tests.kernel_resources import kernels


@pytest.fixture(scope="module")
def found(tmp_path_factory):
    return kernels(tmp_path_factory.mktemp("code"))


def _named(found, *parts):
    sel = {k: v for k, v in found.items() if all(p in k for p in parts)}
    assert sel, parts
    return sel


@pytest.mark.parametrize("metric,sums", [(1, 2), (3, 3)], ids=["l2", "cosine"])
def test_fp16_reference_loads_in_flight(found, metric, sums):
    """Eq. 4 and the cosine against an fp16 reference load 8 groups of both
    arrays before the first sum: 16 loads of 4 registers, beside the fp64
    sums and an address."""
    for name, k in _named(found, f"DriftMetricE{metric}E", "drift_", "EEvPKtPKv").items():
        assert k["vgpr_count"] >= 16 * 4 + 2 * sums + 2, (name, k["vgpr_count"])


def test_batched_live_pass_keeps_to_registers(found):
    """Neither form of the batched live pass keeps its runs' values in LDS or
    scratch, where the compiler puts an array that a loop it did not unroll
    indexes."""
    for name, k in _named(found, "canary_sim_batch_kernel").items():
        assert k["group_segment_fixed_size"] == 0, (name, k)
        assert k["private_segment_fixed_size"] == 0, (name, k)
