"""The replay of test_wait_budget.py for the narrow tiles of single products
whose grid leaves the chip idle and of experts of a few tokens (MXFP4 forward
and dX), and the dispatch's promise that every tile configuration it can launch is one the replay knows."""

import re

import pytest

from test_wait_budget import LATE, configs, replay, source

NARROW = {"fwdc": ["SQ_CFG_FEW_FWDC", "SQ_CFG_MID_FWDC", "SQ_CFG_GROUPED_FEW_FWDC"],
          "dx": ["SQ_CFG_FEW_DX", "SQ_CFG_GROUPED_FEW"]}


@pytest.mark.parametrize("mode,name", [(m, n) for m, names in NARROW.items() for n in names])
def test_waits_cover_every_stage(mode, name):
    cfg = configs()[name]
    for nk in range(1, 41):
        for wave in range(cfg[2] * cfg[3]):
            replay(mode, cfg, nk, wave)


def test_every_launched_configuration_is_replayed():
    used = set(re.findall(r"\bSQ_CFG_\w+", source()))
    known = {n for names in list(LATE.values()) + list(NARROW.values()) for n in names}
    early = {"SQ_CFG_FWD", "SQ_CFG_FEW_FWDR", "SQ_CFG_GROUPED_MID_FWDR"}   # the LDS-dequantised forward waits for every load
    streamed = {"SQ_CFG_DS_STREAM"}
    assert used - known - early - streamed == set()
