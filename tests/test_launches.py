"""What the library launches, and in which order, for calls whose size or place a GPU test does not reach.  Run without a GPU, on a stand-in for the
runtime (launches.c)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

COMMON = r"""
import ctypes as C, sys
import numpy as np
rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2604_10060_amd import binding as b
rt.launch_name.restype = C.c_char_p
rt.launch_grid.restype = C.c_uint
lib = b.load_library()
def context(**kw):
    cfg = b.make_config(**{**dict(n_layers=1, n_q_heads=2, n_kv_heads=2, head_dim=64, tokens_per_frame=1, n_clusters=4, top_k=2, kv_dtype="fp32"), **kw})
    n = b.workspace_size(cfg)
    mem = np.empty(n + 256, np.uint8)               # (no kernel touches it)
    cfg.dev_arena = (mem.ctypes.data + 255) // 256 * 256
    cfg.dev_arena_bytes = n
    h = C.c_void_p()
    assert lib.mosaic_create(C.byref(cfg), C.byref(h)) == b.OK, lib.mosaic_last_error(None)
    return h, mem
x = np.zeros(64, np.uint8)
p = (x.ctypes.data + 15) // 16 * 16                 # (no kernel reads it)
def ok(rc, h): assert rc == b.OK, (rc, lib.mosaic_last_error(h))
def launched():
    names = ["k_set_view", "k_store_visual_assign", "k_store_summary", "k_visual_assign", "k_lloyd_assign", "k_retrieve", "k_assign"]
    out = []
    for i in range(rt.launches()):
        n = rt.launch_name(i).decode()
        out.append((next((k for k in names if k in n), n), tuple(rt.launch_grid(i, d) for d in range(3))))
    rt.forget_launches()
    return out
"""

# A call's frames decided beside their page stores are one launch, as many as it can hold; from there on the call takes launches that can
NESTED = r"""
U = 112
least = (2 ** 22 + U - 1) // U                      # frames whose pages need 2^32 threads in one dimension
h, mem = context(n_layers=28, n_q_heads=4, n_kv_heads=4, max_frames=2 * least + 20, warmup_frames=4, n_partitions=2, visual_dim=8)
ok(lib.mosaic_ingest_frame_visual(h, p, p, p, 4), h)
launched()
ok(lib.mosaic_ingest_frame_visual(h, p, p, p, least - 1), h)
assert [l for l in launched() if l[0] in ("k_store_visual_assign", "k_store_summary", "k_visual_assign")] == \
    [("k_store_visual_assign", (1 + 2 * U * (least - 1), 1, 1))]
ok(lib.mosaic_ingest_frame_visual(h, p, p, p, least), h)
got = [l for l in launched() if l[0] in ("k_store_visual_assign", "k_store_summary", "k_visual_assign")]
assert got == [("k_store_summary", (U, 32768, 2)), ("k_store_summary", (U, least - 32768, 2)), ("k_visual_assign", (1, 1, 1))], got
ok(lib.mosaic_destroy(h), h)
print("OK")
"""


# The views that kernels read are written before the first launch.  A call in a capture records the writes and leaves them to be done again: the next call
# outside may come before the graph's first launch
CAPTURE = r"""
h, mem = context(max_frames=20, warmup_frames=10)
assert rt.launches() == 0
rt.set_capturing(1)
for _ in range(2):
    ok(lib.mosaic_ingest_frame(h, p, p, 3), h)
    assert [l[0] for l in launched()][:3] == ["k_set_view", "k_set_view", "k_store_summary"]
rt.set_capturing(0)
ok(lib.mosaic_ingest_frame(h, p, p, 5), h)
assert [l[0] for l in launched()][:3] == ["k_set_view", "k_set_view", "k_store_summary"]
ok(lib.mosaic_ingest_frame(h, p, p, 1), h)
assert "k_set_view" not in [l[0] for l in launched()]
ok(lib.mosaic_retrieve(h, 0, p, 1), h)
got = [l[0] for l in launched()]
assert got == ["k_retrieve"], got
ok(lib.mosaic_destroy(h), h)
print("OK")
"""


@pytest.mark.parametrize("script", [pytest.param(NESTED, id="nested_call_of_many_frames"), pytest.param(CAPTURE, id="first_call_in_a_capture")])
def test_launches(tmp_path, script):
    so = str(tmp_path / "launches.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launches.c")])
    env = dict(os.environ, LD_PRELOAD=so, PYTHONPATH=os.path.dirname(HERE))
    p = subprocess.run([sys.executable, "-c", COMMON + script, so], env=env, capture_output=True, text=True, timeout=120, cwd=os.path.dirname(HERE))
    assert p.returncode == 0 and p.stdout.strip().endswith("OK"), p.stdout + p.stderr
