"""After a reset the context sizes matching work items by the call again, as a fresh one does: seen
in the cached graphs, which are kept by everything that the launches depend on."""
import numpy as np
import pytest
import torch

from paper_2604_07980_amd import autotune, synth

pytestmark = pytest.mark.gpu


def test_reset_context_is_as_fresh(lib):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    left = torch.randint(0, 256, (1080, 1920), dtype=torch.uint8, device="cuda:0", generator=gen)
    right = torch.roll(left, -9, 1).contiguous()
    n = 150                                      # 311 M boxes x pixels: two groups per wave
    rng = np.random.default_rng(2)
    x0, y0 = rng.integers(0, 1800, n), rng.integers(0, 1000, n)
    side = rng.integers(16, 120, (n, 2))
    boxes = torch.from_numpy(np.stack([x0, y0, x0 + side[:, 0], y0 + side[:, 1], np.ones(n, int)], 1)
                             .astype(np.int32)).cuda()
    p = synth.base_params()
    ws, out = lib.Workspace(), torch.empty((n, 8), dtype=torch.int32, device="cuda:0")

    def builds():
        before = lib.graph_stats()[1]
        lib.range_frame(left, right, boxes, p, workspace=ws, out=out)
        return lib.graph_stats()[1] - before

    autotune.reset(p)
    lib.set_graph(True)
    try:
        assert builds() == 1 and builds() == 0
        want = out.cpu()
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 1)
        assert builds() == 1                     # another size
        assert (out.cpu() == want).all()
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 2)
        assert builds() == 0                     # the size that the call has by itself
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 5)
        autotune.reset(p)
        assert builds() == 0
        assert (out.cpu() == want).all()
        for bad in (-1, 9):
            with pytest.raises(lib.OcsrError):
                lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, bad)
    finally:
        lib.set_graph(False)
        autotune.reset(p)
