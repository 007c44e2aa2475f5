"""What mx_batch_init times: a batch whose grouped schedule runs on register
tiles has the persistent one alone to tune."""
import pytest

from paper_1907_13088_amd import mx

from gpu_helpers import log

pytestmark = pytest.mark.gpu


def _init(n, ng, dtype, path, monkeypatch):
    import time
    import torch
    monkeypatch.setenv("MX_TUNE_CACHE", str(path))
    cfgs = [mx.make_config(2, n, 0.35, (1.0, 1.0), dtype, mx.MX_ALL, 20, 0.0, 0)] * ng
    t0 = time.perf_counter()
    b = mx.Batch(cfgs)
    torch.cuda.synchronize()
    t = time.perf_counter() - t0
    plans = [b.schedule(p) for p in (False, True)]
    b.close()
    return plans, [int(v) for v in path.read_text().split()[-6:]], t


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_a_batch_on_register_tiles(tmp_path, monkeypatch, dtype):
    plans, line, t = _init((150, 90), 6, dtype, tmp_path / "plans.txt", monkeypatch)
    log(f"{dtype}: {plans}, init {t * 1e3:.1f} ms")
    # the grouped schedule is left as it starts; the persistent one is tuned, kept and found again
    assert (plans[0]["sweeps_per_pass"], plans[0]["chunk_rows"], plans[0]["front_rows"]) == (5, 64, 64)
    assert line[:3] == [5, 64, 64]
    assert line[3:] == [plans[1]["sweeps_per_pass"], plans[1]["front_rows"], plans[1]["chunk_rows"]]
    again, _, t2 = _init((150, 90), 6, dtype, tmp_path / "plans.txt", monkeypatch)
    assert again == plans and t2 < t


def test_a_larger_batch(tmp_path, monkeypatch):
    plans, line, _ = _init((1200, 1000), 4, "f32", tmp_path / "plans.txt", monkeypatch)
    assert line == [plans[p][k] for p in (0, 1) for k in ("sweeps_per_pass", "front_rows", "chunk_rows")]
    assert 4 <= plans[0]["sweeps_per_pass"] <= 7
