"""bench.py's bandwidth of a stage is its traffic over a time that is that traffic's alone."""
import pytest

import bench
from paper_2512_16093_amd import synth
from oracle import sla_oracle as so


@pytest.mark.parametrize("quant", ["int8fp8", "qk_int8", "none"])
@pytest.mark.parametrize("cfg", list(synth.CONFIGS.values()), ids=lambda c: c.name)
def test_stages_that_share_a_launch_have_no_bandwidth(cfg, quant):
    Tq, Tk, _, n_m = so.block_counts(cfg.N, cfg.block_q, cfg.block_k, cfg.topk_ratio, cfg.marginal_ratio)
    got = bench.hbm_stage_bytes(cfg.B * cfg.H, cfg.N, cfg.d, Tq, Tk, n_m, quant)
    assert ("prep_kv" in got) == (Tk > 512 and (quant != "none" or n_m > 0))   # (the selection's launch, sla.h)
    assert ("lin_accumulate" in got) == (n_m > 0)
    tensor = cfg.B * cfg.H * cfg.N * cfg.d
    assert got["pool_stats"] == tensor * (6 if quant == "none" else 7)
    if "prep_kv" in got:
        hz = cfg.B * cfg.H * Tk * 129 * 128 * 2 if n_m > 0 else 0
        assert got["prep_kv"] == tensor * (6 if quant == "int8fp8" else 4) + hz
