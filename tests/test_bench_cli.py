"""bench.py's command-line contract on the CPU: a request for more than one
GPU ends before any device work, with a message and no JSON line; and what its
source hash covers."""
import os
import re
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_several_gpus():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert r.stdout.strip() == ""
    assert "one GPU" in r.stderr and "--gpus 1" in r.stderr


def test_source_hash_follows_every_source_of_the_decode_step(tmp_path, monkeypatch):
    """A counter profile counts as current only while the sources it was taken
    from are unchanged: any file that the decode step's units compile changes
    the hash, and no other kernel's does."""
    sys.path.insert(0, ROOT)
    import bench
    csrc = os.path.join("paper_2607_00760_amd", "csrc")
    shutil.copytree(os.path.join(ROOT, csrc), tmp_path / csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    units = [f for f in sorted(os.listdir(tmp_path / csrc)) if f.startswith("attn_") or f in ("api.hip", "decode.hip", "score.hip")]
    decode = set()
    while units:                                             # with the headers they include
        f = units.pop()
        decode.add(f)
        inc = re.findall(r'^#include "([^"/]+)"', (tmp_path / csrc / f).read_text(), flags=re.M)
        units += [x for x in inc if x not in decode]
    assert {"topk.h", "attn.h", "score.hip", "mosaic_internal.h"} <= decode
    first = bench.source_hash()
    for f in sorted(os.listdir(tmp_path / csrc)):
        path = tmp_path / csrc / f
        text = path.read_text()
        path.write_text(text + "\n")
        assert (bench.source_hash() != first) == (f in decode), f
        path.write_text(text)
    assert bench.source_hash() == first
