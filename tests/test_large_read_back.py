"""Large read-backs go through pieces of pinned memory while helper threads copy them on: every byte arrives, no piece is overwritten
before it has been copied on, and an error leaves nothing under way.  Run without a GPU, on a stand-in for the runtime (pinned_copies.c)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

SCRIPT = r"""
import ctypes as C, sys
import numpy as np
from paper_2604_10060_amd import binding as b
rt = C.CDLL(sys.argv[1])
lib = b.load_library()
rng = np.random.default_rng(5)
# (units, clusters, channels): below the line, at it, one piece and a little, as many pieces as slots, many, and an odd number of units
for L, CL, D in [(2, 60, 64), (8, 256, 128), (9, 256, 128), (16, 512, 128), (64, 1000, 128), (7, 601, 64), (33, 777, 128)]:
    cfg = b.make_config(n_layers=L, n_q_heads=1, n_kv_heads=1, head_dim=D, tokens_per_frame=1, max_frames=2 * CL, n_clusters=CL, top_k=1,
                        kv_dtype="fp32", warmup_frames=CL, max_q_tokens=1)
    n = b.workspace_size(cfg)
    mem = rng.integers(0, 256, n + 256, dtype=np.uint8)
    cfg.dev_arena = (mem.ctypes.data + 255) // 256 * 256
    cfg.dev_arena_bytes = n
    h = C.c_void_p()
    assert lib.mosaic_create(C.byref(cfg), C.byref(h)) == b.OK, lib.mosaic_last_error(None)
    x = np.zeros(64, np.uint8)
    p = (x.ctypes.data + 15) // 16 * 16
    assert lib.mosaic_ingest_frame(h, p, p, CL) == b.OK
    size = L * CL * D * 8
    for rep in range(3):
        rt.copies(); rt.most_open()
        r = np.zeros(size, np.uint8)
        assert lib.mosaic_get_centroids(h, r.ctypes.data, None) == b.OK
        at = mem.tobytes().find(r[:256].tobytes())
        assert at >= 0 and (mem[at:at + size] == r).all(), (L, CL, D)
        sent = rt.copies()
        assert sent == (0 if size < 2 << 20 else -(-size // (2 << 20))) and rt.most_open() <= 4
    if size > 12 << 20:
        for bad in (0, 2, 5):                        # a copy that is refused: an error, and the next read-back is whole again
            rt.copies(); rt.fail_copy(bad)
            assert lib.mosaic_get_centroids(h, r.ctypes.data, None) == b.EHIP
            rt.fail_copy(-1); rt.copies()
            r[:] = 0
            assert lib.mosaic_get_centroids(h, r.ctypes.data, None) == b.OK
            assert (mem[at:at + size] == r).all()
    assert lib.mosaic_destroy(h) == b.OK
print("OK")
"""


def test_large_read_backs_through_pinned_pieces(tmp_path):
    so = str(tmp_path / "pinned_copies.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "pinned_copies.c")])
    env = dict(os.environ, LD_PRELOAD=so, PYTHONPATH=os.path.dirname(HERE))
    p = subprocess.run([sys.executable, "-c", SCRIPT, so], env=env, capture_output=True, text=True, timeout=120, cwd=os.path.dirname(HERE))
    assert p.returncode == 0 and p.stdout.strip().endswith("OK"), p.stdout + p.stderr
