"""Resources the compiler must give some kernels for them to run as they are
written: what a source line alone does not show (CPU only)."""
import pytest

from tests.kernel_resources import kernels, most_loads_without_a_wait


@pytest.fixture(scope="module")
def found(tmp_path_factory):
    return kernels(tmp_path_factory.mktemp("code"))


def _named(found, *parts):
    sel = {k: v for k, v in found.items() if all(p in k for p in parts)}
    assert sel, parts
    return sel


@pytest.mark.parametrize("kernel", ["drift_partial_kernel", "drift_team_kernel"])
@pytest.mark.parametrize("metric,loads", [(0, 24), (1, 16), (2, 24), (3, 16)],
                         ids=["l2", "l2_f16", "cosine", "cosine_f16"])
def test_block_reductions_load_a_step_before_its_sums(tmp_path, kernel, metric, loads):
    """Eq. 4 and the cosine load 8 groups of a thread (16 bytes of activations
    each, and 32 of an fp32 or 16 of an fp16 reference) before they wait for
    the first."""
    found = most_loads_without_a_wait(tmp_path, kernel)
    runs = {k: v for k, v in found.items() if f"DriftMetricE{metric}E" in k}
    assert runs
    assert all(v >= loads for v in runs.values()), runs


def test_batched_live_pass_keeps_to_registers(found):
    """Neither form of the batched live pass keeps its runs' values in LDS or
    scratch, where the compiler puts an array that a loop it did not unroll
    indexes."""
    for name, k in _named(found, "canary_sim_batch_kernel").items():
        assert k["group_segment_fixed_size"] == 0, (name, k)
        assert k["private_segment_fixed_size"] == 0, (name, k)
