"""The form of the band operator (spectral or direct) in the autotuner's caches:
a choice made on a full card or under a switch that fixes the form does not
outlive it."""
import pytest

import synth
from gpu_common import leave_free, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def tune_file(tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("PSOAM_TUNE_CACHE", str(path))
    monkeypatch.delenv("PSOAM_SPECTRAL", raising=False)
    return path


def _tuned(cfg, t0, taps, phi, sp, prec):
    import paper_2510_23739_amd as pk
    p = pk.Plan.from_config(cfg, phi, sp, t0, taps, prec=prec, tune=True)
    out = p.stats()["spectral"], p.tune_report
    p.close()
    say(f"[tune form] {cfg.nx}x{cfg.ny}x{cfg.nz} {prec}: {out}")
    return out


def _big(seed):
    """Much faster in the spectral form."""
    cfg = synth.Config("t", nx=60, ny=60, nz=48, n_species=2, n_pulses=16, nt=160, f=21, k1=1, seed=seed)
    t0, taps = synth.sir_table(cfg.nz, cfg.f, cfg.nt)
    return cfg, t0, taps * (1.0 + 0.01 * seed), synth.phi_depth(cfg.nz), synth.species(2)


def test_a_full_card_decides_nothing_for_later(tune_file, monkeypatch):
    torch = torch_cuda()
    import paper_2510_23739_amd as pk
    problem = _big(1)
    torch.cuda.empty_cache()
    plan = pk.Plan.from_config(problem[0], *problem[3:], *problem[1:3], prec="fp32")
    need = plan.stats()["spectral_bytes"]
    plan.close()
    say(f"[tune form] spectra and tables: {need} bytes")
    # a third of what is left is less than the spectra
    rest = leave_free(torch, 2 * need)
    if rest is None:
        pytest.skip("the card is in use")
    form, rep = _tuned(*problem, "fp32")
    del rest
    torch.cuda.empty_cache()
    assert form == 0
    assert not tune_file.exists() or tune_file.read_text() == ""
    assert _tuned(*problem, "fp32")[0] == 1               # this process's cache: shapes, not the form
    monkeypatch.setenv("PSOAM_TUNE_MEMO", "0")
    form, rep = _tuned(*problem, "fp32")                   # a new process's
    assert form == 1 and rep["from_cache"] == 0


def test_a_forced_form_is_not_kept(tune_file, monkeypatch):
    torch_cuda()
    problem = _big(2)
    monkeypatch.setenv("PSOAM_SPECTRAL", "0")
    assert _tuned(*problem, "bf16_split")[0] == 0
    monkeypatch.delenv("PSOAM_SPECTRAL")
    form, rep = _tuned(*problem, "bf16_split")
    assert form == 1 and rep["from_cache"] == 0
    # (timed against the direct form this time, and kept)
    monkeypatch.setenv("PSOAM_TUNE_MEMO", "0")
    form, rep = _tuned(*problem, "bf16_split")
    assert form == 1 and rep["from_cache"] == 2
