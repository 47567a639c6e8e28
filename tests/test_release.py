"""The memory that the library keeps of released matrices can be given back
through the binding."""
import pytest


def test_release_without_a_matrix():
    from paper_1307_6209_amd import sellcs
    sellcs.sell_destroy(None)


@pytest.mark.gpu
def test_kept_memory_is_given_back():
    import torch

    import synth
    from gpu_util import build
    from paper_1307_6209_amd import sellcs

    sellcs.sell_destroy(None)
    h = build(synth.stencil27(60), 32, 1)
    held = h.info["device_bytes"]
    assert held > 64 << 20
    sellcs.sell_destroy(h)
    kept = torch.cuda.mem_get_info()[0]
    sellcs.sell_destroy(None)
    assert torch.cuda.mem_get_info()[0] - kept >= held
