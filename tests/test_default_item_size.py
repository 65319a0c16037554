"""The size of matching work items by a call's own size is the library's default, which the tuner
starts from, tries and restores. Host side; the GPU side is in test_gpu_default_item_size.py."""
import numpy as np
import pytest

from paper_2604_07980_amd import autotune, ocsr


@pytest.fixture
def options(monkeypatch):
    """The options that the library was given last, and every value each was given."""
    state, seen = {}, {}

    def set_option(o, v, device=None):
        state[o] = v
        seen.setdefault(o, []).append(v)

    monkeypatch.setattr(autotune.ocsr, "set_option", set_option)
    monkeypatch.setattr(autotune.ocsr, "set_variant", lambda *a: None)
    monkeypatch.setattr(autotune.ocsr, "variant_candidates", lambda bw, bh, nd: [])
    monkeypatch.setattr(autotune, "path_shapes", lambda params: [(8, 8, 96)])
    monkeypatch.setattr(autotune, "_arch", lambda: "gfx950")
    monkeypatch.setattr(autotune, "_snapshot", lambda r: r)
    return state, seen


def test_reset_restores_the_size_by_call(options):
    state, _ = options
    autotune.apply(autotune.Table(arch="gfx950", blocks_per_wave=4))
    assert state[ocsr.OPTION_BLOCKS_PER_WAVE] == 4
    autotune.reset({})
    assert state[ocsr.OPTION_BLOCKS_PER_WAVE] == 0
    autotune.apply(autotune.Table(arch="gfx950"))
    assert state[ocsr.OPTION_BLOCKS_PER_WAVE] == 0


@pytest.mark.parametrize("best", [0, 1, 3])
def test_tune_tries_the_default_and_every_size_it_takes(options, monkeypatch, best):
    state, seen = options
    monkeypatch.setattr(autotune, "_time_ms", lambda run, reps, warmup:
                        1.0 - 0.1 * (state[ocsr.OPTION_BLOCKS_PER_WAVE] == best))
    table = autotune.tune(lambda: np.zeros(4), {}, reps=1, warmup=0)
    assert {0, 1, 2, 3} <= set(seen[ocsr.OPTION_BLOCKS_PER_WAVE])
    assert seen[ocsr.OPTION_BLOCKS_PER_WAVE][0] == 0
    assert table.blocks_per_wave == best and state[ocsr.OPTION_BLOCKS_PER_WAVE] == best
    assert autotune.from_json(autotune.to_json(table)) == table


@pytest.mark.parametrize("value", [-1, 9])
def test_tables_refuse_other_sizes(value):
    with pytest.raises(ValueError):
        autotune.from_json('{"arch": "gfx950", "variants": {}, "blocks_per_wave": %d, "match_wgs_per_cu": 16}' % value)
