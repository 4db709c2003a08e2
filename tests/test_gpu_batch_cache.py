"""Lines of a tuner's cache file from before the tiles: their key hashes the cavity shapes alone and
their last two numbers are rows and strips of another kernel.  They are left alone and the batch is
tuned: the file gains a line, which the next batch uses."""
import pytest
import torch

from paper_1308_2071_amd import Batch, workloads

pytestmark = pytest.mark.gpu


def old_key(params, dtype):
    h = 1469598103934665603
    for v in [len(params)] + [n for p in params for n in (p["nx"], p["ny"])]:
        for k in range(8):
            h = ((h ^ (v >> 8 * k & 0xff)) * 1099511628211) % 2 ** 64
    arch = torch.cuda.get_device_properties(0).gcnArchName.replace(":", "_").replace(" ", "_")
    return f"v3|{arch}|{dtype}|{h:016x}|s0"


@pytest.mark.parametrize("last", ["3 1", "12 4", "0 1"])
def test_lines_of_another_set_of_tiles_are_tuned_anew(last, tmp_path):
    params = [workloads.cavity(n, n + 3, Ra=1e4, Pr=0.71, Da=1e-2, dtype="fp32")
              for n in (40, 64, 90)]
    path = tmp_path / "tune.txt"
    line = f"{old_key(params, 'fp32')} 4 1 0 {last}\n"
    path.write_text(line)
    b = Batch(params, [0.5] * 3, tune_cache_path=str(path))
    lines = path.read_text().splitlines(keepends=True)
    assert len(lines) == 2 and lines[0] == line
    assert lines[1].split()[0] != line.split()[0]
    again = Batch(params, [0.5] * 3, tune_cache_path=str(path))
    assert again.shape() == b.shape()
    assert len(path.read_text().splitlines()) == 2
    again.close()
    b.close()
