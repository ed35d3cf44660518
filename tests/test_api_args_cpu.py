"""Arguments that the Python wrappers refuse before a call: a variant or a
split that is no whole number is a TypeError, not AUTO or no split."""
import pytest

from paper_2608_03057_amd import api


@pytest.mark.parametrize("variant,split_k", [(None, 0), (0.0, 0), ("", 0), (0, None), (0, 0.0)])
def test_opts_refuse_other_types(variant, split_k):
    with pytest.raises(TypeError):
        api._opts(variant, None, None, split_k)


def test_opts_defaults():
    o = api._opts(0, None, None, 0)
    assert (o.variant, o.split_k, o.workspace_bytes) == (0, 0, 0)
    assert not o.W_planes and not o.workspace and not o.W_packed and not o.act_params
