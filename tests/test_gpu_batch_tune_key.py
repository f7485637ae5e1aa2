"""A workgroup size recorded by a library that scheduled the tubes in another way is
not taken: the record names the schedule it was timed with.
"""
import pytest
import torch

import paper_1210_5246_amd as csh
import workloads as wl

pytestmark = pytest.mark.gpu


def test_a_record_of_another_schedule_is_not_taken(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("CSH_TUNE_CACHE", str(cache))
    t = wl.tubes(ntubes=24, seed=41)
    print("autotune key", flush=True)
    W = torch.from_numpy(t.W).cuda()
    csh.Batch(W, t.offsets).autotune(probe_steps=2)
    key = cache.read_text().splitlines()[0].rsplit(" ", 1)[0]
    first, rest = key.split(";", 1)
    # a record without a schedule (as libraries wrote before it was in the key) and one of another schedule
    p = torch.cuda.get_device_properties(0)
    bare = f"arch={p.gcnArchName};cus={p.multi_processor_count};tubes=24;cells={int(t.offsets[-1])};" \
           f"maxlen={int(t.lengths.max())}"
    for old in (bare, f"schedule=1;{bare}"):
        cache.write_text(f"{old} 64\n")
        best = csh.Batch(W, t.offsets).autotune(probe_steps=2)
        assert cache.read_text().splitlines() == [f"{old} 64", f"{key} {best}"]  # probed and recorded
    assert first.startswith("schedule=") and rest == bare
