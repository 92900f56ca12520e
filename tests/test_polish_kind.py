"""Which polish runs, as the library reports it (device-free), at the limits that
bodex_qp.h states; and the autotuner times a polish once however many values of
polish_chunk select it."""
import ctypes

import pytest

from paper_2412_16490_amd import api, autotune
from paper_2412_16490_amd import workload as wl


def _kind(n_qps=131072, **kw):
    return api.bodex_qp_polish_kind(api.default_params(**kw), n_qps)


def test_pyramid():
    assert _kind() == _kind(1) == _kind(polish_chunk=1) == _kind(polish_chunk=24) == "newton"
    assert _kind(polish_chunk=0) == "one-lane" and _kind(gamma=0.5) == "one-lane"
    assert _kind(eps_reg=5e-7) == "newton" and _kind(eps_reg=4e-7) == "chunked"
    assert _kind(polish_steps=32) == "newton" and _kind(polish_steps=31) == "chunked"
    assert _kind(eps_reg=4e-7, polish_chunk=0) == "one-lane"
    assert _kind(flags_clear=api.F_POLISH) == "none"


def test_cone():
    cone = dict(friction_cone=api.CONE_CIRCULAR)
    assert _kind(8192, **cone) == "newton" and _kind(8193, **cone) == "barrier"
    assert _kind(100, polish_chunk=0, **cone) == _kind(100, gamma=0.5, **cone) == "barrier"
    assert _kind(100, eps_reg=4e-7, **cone) == "barrier" and _kind(100, flags_clear=api.F_POLISH, **cone) == "none"
    assert _kind(100, polish_steps=6, **cone) == "newton" and _kind(100, polish_steps=0, **cone) == "barrier"


def test_bad_parameters():
    for p, n in ((api.default_params(m_max=0), 10), (api.default_params(), -1)):
        with pytest.raises(api.BodexError):
            api.bodex_qp_polish_kind(p, n)


@pytest.mark.parametrize("kw,runs", [({}, 12), (dict(eps_reg=4e-7), 48), (dict(gamma=0.5), 6)])
def test_autotuner_times_a_polish_once(monkeypatch, kw, runs):
    import torch
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda *a: "none")
    monkeypatch.setattr(torch.cuda, "Stream", lambda *a: None)
    monkeypatch.setattr(autotune, "_time_solve", lambda p, batch, reps, stream: (1e-3, True))
    b = wl.uniform_batch(1, 4, 5, 16)
    best, table = autotune.tune(b, base=api.default_params(**kw), cache_path=None)
    assert len(table) == runs and best in [t["knobs"] for t in table]
