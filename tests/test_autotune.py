"""The autotuner's cache entry of a set of subgrids for which the library's
default is the fastest candidate."""
import torch


def test_cached_default_is_not_tuned_again(tmp_path, monkeypatch):
    from paper_1804_10120_amd import autotune
    monkeypatch.setenv("TLMI_TUNE_CACHE", str(tmp_path / "tune.json"))
    doms = [{"K": torch.empty(6, n)} for n in (512, 1000)]
    tuned = []
    monkeypatch.setattr(autotune, "tune_plan",
                        lambda *a, **k: tuned.append(k) or {"tune": {"block": 64}})
    assert autotune.plan_tune(doms) == {"block": 64} and len(tuned) == 1
    autotune.save_cache({autotune.plan_key(doms): {"tune": None, "us": 1.0}})
    assert autotune.plan_tune(doms) is None and len(tuned) == 1
    assert autotune.lookup_plan(doms) is None
