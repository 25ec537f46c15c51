"""The benchmark's line reports a measured HBM traffic only while the device
code is the one it was measured on."""

import json
import os
import shutil

import bench


def test_traffic_is_dropped_when_any_kernel_source_changes(tmp_path, monkeypatch):
    csrc, profiles = tmp_path / "csrc", tmp_path / "profiles"
    shutil.copytree(bench.CSRC, csrc)
    profiles.mkdir()
    monkeypatch.setattr(bench, "CSRC", str(csrc))
    monkeypatch.setattr(bench, "PROFILES", str(profiles))
    with open(profiles / "traffic_mix_multirate_c1_f16.json", "w") as f:
        json.dump({"kernel_sha": bench.kernel_hash(), "hbm_bytes_per_launch": 17}, f)
    assert bench.load_traffic("mix", "f16") == 17
    sources = [n for n in os.listdir(csrc) if n.endswith((".hip", ".h"))]
    assert {"lloid_kernels.hip", "lloid_mix.hip", "lloid_device.h"} <= set(sources)
    for name in sources:
        text = (csrc / name).read_text()
        (csrc / name).write_text(text + "\n")
        assert bench.load_traffic("mix", "f16") is None, name
        (csrc / name).write_text(text)
        assert bench.load_traffic("mix", "f16") == 17
