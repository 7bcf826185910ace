"""CPU check of bench.py's legs that apply a fused program by one call: its
blocks share sweeps, so a leg's figure is the time, not the blocks' number as
bytes over the time.  The library, torch and the events are stand-ins."""
import os
import sys
from unittest.mock import MagicMock

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import workloads as W  # noqa: E402


def _stand_ins():
    P, torch, H = MagicMock(), MagicMock(), MagicMock()
    P.fuse.return_value.count = 52
    P.fuse.return_value.blocks.return_value = []
    P.gate_entries.return_value = [((0,), None, (), None, False)] * 90
    torch.cuda.Event.return_value.elapsed_time.return_value = 1.0
    return P, torch, H


def _keys(v):
    return {k for k in v} | {k for x in v.values() if isinstance(x, dict) for k in _keys(x)}


def test_seeds_report_times():
    P, torch, H = _stand_ins()
    out = bench.seeds_leg(P, W, torch, H, 12, 2, 5, 3)
    assert out["c64"]["mean_ms"] == 1.0
    assert not any("GBps" in k or "frac" in k for k in _keys(out))


def test_fusion_widths_report_times():
    P, torch, H = _stand_ins()
    out = bench.kmax_leg(P, W, torch, H, W.brickwork(12, 2, 0), 12)
    for dt in ("c64", "c128"):
        assert "GBps" in out[dt]["unfused"]  # a sweep a gate
        for k in ("kmax4", "kmax5", "kmax6"):
            assert out[dt][k]["apply_ms"] == 1.0 and "GBps" not in out[dt][k]


def test_fused_qft_reports_times():
    P, torch, H = _stand_ins()
    out = bench.diagonal_leg(P, W, torch, H, 12, 1)
    for dt in ("c64", "c128"):
        assert "GBps" in out[dt]["diag_k2"]
        for k in ("qft_dense_only", "qft_dense_and_diagonal", "qft_coupled"):
            assert out[dt][k]["apply_ms"] == 1.0 and "GBps" not in out[dt][k]


def test_batch_reports_no_bandwidth():
    with open(os.path.join(ROOT, "bench.py")) as f:
        assert "effective_GBps" not in f.read()
