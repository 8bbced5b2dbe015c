"""Host side of sm_attn_block's workspace, without a GPU."""
import ctypes as C
import pytest
from paper_2404_13528_amd import binding as sm


def workspace(kind, B, S, E, heads, F, mode=sm.SM_ELIDED):
    c = sm.AttnCfg(kind, sm.SM_BF16, B, S, E, heads, F, 0, 0, 32, 0, 0, 10000.0, 1e-5, 1e-6)
    return sm.lib().sm_attn_block_workspace_bytes(C.byref(c), mode)


@pytest.mark.parametrize("shape", [(0, 1, 333, 4096, 32, 11008), (0, 1, 701, 2048, 16, 5632), (2, 2, 577, 1024, 16, 4096), (0, 1, 333, 1024, 8, 2816)])
def test_the_size_depends_on_the_configuration_alone(shape):
    """A program that sweeps tiles (sm_gemm_tuning) after or before it asked needs the same workspace."""
    n = workspace(*shape)
    assert n > 0
    try:
        sm.gemm_tuning(64, 2)
        assert workspace(*shape) == n
    finally:
        sm.gemm_tuning(0, 0)
