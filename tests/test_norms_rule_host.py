"""Which calls take their value norms beside the scan's first pass (host code: no GPU). One workgroup per CU at most: beyond that two
workgroups of the scan alone share a CU where rows are short, and the ends of a launch weigh more with eight waves than with four."""
import pytest

from paper_2602_08686_amd import binding as B
from parity_util import norms_beside_the_scan
from test_gpu_norms_in_scan import GROUPS, LENGTHS, WIDTHS


def params(batch, kv, group, window, d, T, dtype="bf16", flags=B.FLAG_VALUE_NORM):
    return B.make_params(batch=batch, n_q_heads=kv * group, n_kv_heads=kv, head_dim=d, seq_len=T, window=window, dtype=dtype,
                         pool=B.POOL_AVG, pool_kernel=7, budget=window + 8, cap=T, flags=flags)


@pytest.mark.parametrize("batch,kv,group,window,d,T", [
    (1, 8, 1, 32, 128, 16384), (4, 8, 4, 32, 128, 10006), (16, 8, 4, 32, 128, 32768), (16, 8, 4, 32, 64, 16384), (1, 32, 1, 32, 128, 4096),
    (2, 8, 2, 64, 64, 33000)])
def test_up_to_one_workgroup_per_cu(batch, kv, group, window, d, T):
    p = params(batch, kv, group, window, d, T)
    assert norms_beside_the_scan(p) and not norms_beside_the_scan(p, lse_given=True)
    assert not norms_beside_the_scan(params(batch, kv, group, window, d, T, dtype="f32"))
    assert not norms_beside_the_scan(params(batch, kv, group, window, d, T, flags=0))


@pytest.mark.parametrize("batch,kv,group,window,d,T", [
    (32, 32, 4, 32, 64, 2888), (32, 32, 4, 32, 64, 4733), (16, 8, 1, 32, 64, 33000), (24, 8, 3, 32, 128, 14629), (24, 8, 1, 32, 128, 18237),
    (24, 32, 4, 32, 64, 1552)])
def test_not_in_launches_of_more_workgroups(batch, kv, group, window, d, T):
    assert not norms_beside_the_scan(params(batch, kv, group, window, d, T))


def test_the_comparison_on_the_gpu_has_both_kinds():
    """test_gpu_norms_in_scan compares a call with one that always takes the separate kernel: most of its shapes must not."""
    for d in WIDTHS:
        for group, window in GROUPS:
            beside = sum(norms_beside_the_scan(params(1, kv, group, window, d, T)) for kv, T in LENGTHS)
            assert beside == 0 if group * ((window + 31) // 32) > 4 else 3 <= beside < len(LENGTHS), (d, group, window, beside)
