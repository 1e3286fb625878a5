"""bench.py --write-traffic: the counter files' rows of the kernel instance that a workload's pass runs."""

import csv
import json

import pytest

import bench


# workload, 16-row blocks of its pass's kernel instance (1, 2, 3, 4, 6 or 8)
@pytest.mark.parametrize("workload,blocks", [("llama30b_p1024_n8", 1), ("llama7b_p512_n31", 2),
                                             ("llama7b_p2048_n41", 3), ("llama13b_p1024_n41", 3),
                                             ("llama7b_p512_n128", 8)])
def test_instance_of_the_workload(tmp_path, monkeypatch, capsys, workload, blocks):
    # every instance in the files, each with values of its own: fetch 1000 MB, write MB (KiB)
    files = []
    for name, scale in (("fetch", 1000), ("write", 1)):
        path = tmp_path / f"{name}.csv"
        with open(path, "w", newline="") as f:
            w = csv.writer(f)
            w.writerow(["Kernel_Name", "Counter_Value"])
            w.writerow(["FillFunctor<float>", 1048576])
            w.writerow(["__amd_rocclr_copyBuffer", 16384 if name == "fetch" else 32768])
            for mb in (1, 2, 3, 4, 6, 8):
                for _ in range(3):
                    w.writerow([f"pass_kernel<{mb}, 128, false>(llmcad::PassParams)", scale * mb])
        files.append(str(path))
    out = tmp_path / "traffic.json"
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(out))
    bench.write_traffic(*files, workload, 1024)
    capsys.readouterr()
    entry = json.loads(out.read_text())[workload]
    assert f"pass_kernel<{blocks}, 128" in entry["kernel"]
    assert entry["read_bytes"] == 2 * 1000 * blocks * 1024 and entry["write_bytes"] == blocks * 1024
