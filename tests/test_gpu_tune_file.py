"""The tuning cache file: choices are read back for the same model and size; lines without the kernels'
revision, of another one or with a variant that does not exist are passed over."""
import numpy as np
import pytest
import torch

import synthetic as sy

pytestmark = pytest.mark.gpu

WATER = sy.model_config("water")


def test_lines(tmp_path, monkeypatch):
    import paper_2604_21441_amd as P
    path = tmp_path / "tuned"
    w = sy.flat_weights(sy.model_weights(WATER, seed=1))
    pos, Z, box = sy.water_box(64, 12.42, seed=0)
    d = torch.from_numpy(pos).cuda()

    def variants(tune=False):
        m = P.NNPModel(WATER, weights=w)
        m.compute(d, Z, box)
        out = m.autotune(2) if tune else m.variants()
        m.close()
        return out

    default = variants()
    monkeypatch.setenv("NNP_TUNE_CACHE", str(path))
    tuned = variants(tune=True)
    lines = path.read_text().splitlines()
    fields = [l.split() for l in lines]
    arch = {f[0] for f in fields}
    assert len(arch) == 1 and all(len(f) == 6 for f in fields)
    assert variants() == tuned
    name, revision = arch.pop().split("/")
    assert name == torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    network = [f for f in fields if f[3] == "2"][0]
    other = "1" if default["network"] != 1 else "2"

    def with_network(arch, variant):
        path.write_text(" ".join([arch] + network[1:5] + [variant]) + "\n")
        return variants()["network"]

    assert with_network(f"{name}/{revision}", other) == int(other)
    assert with_network(name, other) == default["network"]
    assert with_network(f"{name}/{int(revision) - 1}", other) == default["network"]
    assert with_network(f"{name}/{revision}", "99") == default["network"]
    assert with_network(f"{name}/{revision}", "-1") == default["network"]
