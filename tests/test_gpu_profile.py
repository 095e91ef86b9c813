"""Event timing of the passes (kb_profile_enable / kb_profile_select): every
phase records one bracket per launch group, a phase mask records only the
phases it names, and recording off records nothing."""
import ctypes

import pytest

import kbgen
from gpu_util import to_em

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2002_06115_amd as kbf
    w = kbgen.METAQA.scaled(20_000, 150_000, batch=32, tag=5)
    kb = kbgen.make_kb(w)
    gkb = kbf.KB(kb.subj, kb.rel, kb.obj, w.n_entities, w.n_relations)
    X, R, dY = to_em(kbgen.make_x(w)), to_em(kbgen.make_r(w)), to_em(kbgen.make_dy(w))
    yield kbf, gkb, X, R, dY
    gkb.close()


def step(gkb, X, R, dY):
    import torch
    gkb.follow(X, R)
    gkb.follow_backward(X, R, dY)
    torch.cuda.synchronize()


def test_all_phases(setup):
    kbf, gkb, X, R, dY = setup
    gkb.profile(True)
    step(gkb, X, R, dY)
    ph = gkb.profile_read()
    gkb.profile(False)
    info = gkb.info()
    for i, p in enumerate(("fwd", "dx", "dr")):
        ms, n = ph[f"{p}_stream"]
        assert n == 1 and ms > 0, p
        # one bracket around the tail launch, one around the further combine levels
        assert ph[f"{p}_tail"][1] == 1 and ph[f"{p}_combine"][1] == 1, p
        if info["n_levels"][i] > 1:
            assert ph[f"{p}_combine"][0] > 0, p


def test_phase_mask_records_only_named_phases(setup):
    kbf, gkb, X, R, dY = setup
    gkb.profile(True, phases=["dr_stream", "fwd_tail"])
    step(gkb, X, R, dY)
    step(gkb, X, R, dY)
    ph = gkb.profile_read()
    gkb.profile(False)
    assert {p for p, (ms, n) in ph.items() if n} == {"dr_stream", "fwd_tail"}
    assert ph["dr_stream"][1] == 2 and ph["dr_stream"][0] > 0


def test_off_records_nothing_and_bits_past_the_phases_are_ignored(setup):
    kbf, gkb, X, R, dY = setup
    gkb.profile(False)
    step(gkb, X, R, dY)
    assert all(n == 0 for ms, n in gkb.profile_read().values())
    lib = ctypes.CDLL(kbf.LIB_PATH)
    lib.kb_profile_select.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    assert lib.kb_profile_select(gkb._handle, 0xFFFFFFFF) == 0
    step(gkb, X, R, dY)
    ph = gkb.profile_read()
    assert all(n == 1 for ms, n in ph.values())
    gkb.profile(False)


@pytest.mark.parametrize("prefill", ["0", "1"])
@pytest.mark.parametrize("b", [2, 10, 32])
def test_tail_phase_follows_the_sweep(b, prefill, monkeypatch):
    """The tail phase names what it launches and counts one launch a pass, with the
    empty rows written one by one or by a sweep, with and without split rows."""
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2002_06115_amd as kbf
    monkeypatch.setenv("KBFOLLOW_PREFILL", prefill)
    n_e, n_r = 500, 4
    g = np.random.default_rng(b)
    # 100 objects and 400 subjects have triples, no row is long; one relation has none.
    o, s, r = np.arange(400) % 100, np.arange(400), np.arange(400) % 3
    few = kbf.KB(s.astype(np.int32), r.astype(np.int32), o.astype(np.int32), n_e, n_r)
    assert few.info()["n_split_rows"][0] == 0 and few.info()["n_split_rows"][2] > 0
    fill = "fill_kernel<false>"
    vec = 4 if b >= 5 else 1
    names = few.phase_kernels(b)
    if prefill == "1":
        assert names["fwd_tail"] == fill
        assert names["dr_tail"].startswith(fill + f" + tail_kernel<{vec}, ")
        assert few.phase_kernels(b, residual=True)["dx_tail"] == "fill_kernel<true>"
    else:
        assert names["fwd_tail"].startswith(f"tail_kernel<{vec}, ")
        assert names["dr_tail"].startswith(f"tail_kernel<{vec}, ")
    X, R, dY = (torch.from_numpy(g.random((n, b), np.float32)).cuda() for n in (n_e, n_r, n_e))
    few.profile(True)
    step(few, X, R, dY)
    step(few, X, R, dY)
    ph = few.profile_read()
    few.profile(False)
    for p in ("fwd", "dx", "dr"):
        assert ph[f"{p}_stream"][1] == 2 and ph[f"{p}_tail"][1] == 2, (p, ph)
        assert ph[f"{p}_tail"][0] > 0
    few.close()
    # Every row of every layout has triples: no sweep whatever the switch says.
    full = kbf.KB(np.arange(60, dtype=np.int32), np.arange(60, dtype=np.int32) % 2,
                  np.arange(60, dtype=np.int32), 60, 2)
    assert full.phase_kernels(b)["fwd_tail"] == ""
    full.close()
