"""The mosaic_get_* observers hand over finished results: the caller's memory is pageable, and an asynchronous copy into
pageable memory is not promised to be over when its stream is.  Run without a GPU, on a stand-in for the runtime
(late_copies.c) whose asynchronous copies never end by themselves."""
import os
import subprocess
import sys



HERE = os.path.dirname(os.path.abspath(__file__))

SCRIPT = r"""
import ctypes as C, sys
import numpy as np
from paper_2604_10060_amd import binding as b
late = C.CDLL(sys.argv[1])
late.copied_bytes.restype = C.c_size_t
lib = b.load_library()
PAT = 0x07
I, D = 0x07070707, np.frombuffer(bytes([PAT] * 8), np.float64)[0]

class Ctx:
    # a context over an arena full of one byte, so that whatever an observer copies out of it is known
    def __init__(self, n_frames, **kw):
        base = dict(n_layers=3, n_q_heads=4, n_kv_heads=2, head_dim=64, tokens_per_frame=2, max_frames=40, n_clusters=8,
                    top_k=4, kv_dtype="fp32", warmup_frames=16)
        self.cfg = b.make_config(**{**base, **kw})
        n = b.workspace_size(self.cfg)
        self.mem = np.full(n + 256, PAT, np.uint8)
        self.cfg.dev_arena = (self.mem.ctypes.data + 255) // 256 * 256
        self.cfg.dev_arena_bytes = n
        self.h = C.c_void_p()
        assert lib.mosaic_create(C.byref(self.cfg), C.byref(self.h)) == b.OK, lib.mosaic_last_error(None)
        x = np.zeros(64, np.uint8)
        p = (x.ctypes.data + 15) // 16 * 16        # (no kernel reads it)
        if self.cfg.n_partitions:
            self.ok(lib.mosaic_ingest_frame_visual(self.h, p, p, p, n_frames))
        else:
            self.ok(lib.mosaic_ingest_frame(self.h, p, p, n_frames))
        self.p = p
    def ok(self, rc):
        assert rc == b.OK, (rc, lib.mosaic_last_error(self.h))

def ints(*s): return np.zeros(s, np.int32)
def dbls(*s): return np.zeros(s, np.float64)
def same(*arrays):
    for a in arrays:
        assert a.size and (a == (I if a.dtype == np.int32 else D)).all(), a.ravel()[:8]
    assert late.late_copies_pending() == 0

U, F, CL = 6, 40, 8
for n in (40, 23):                                   # a full stream, and one with room left
    c = Ctx(n)
    late.copied_bytes()
    a = ints(U, n); c.ok(lib.mosaic_get_assignments(c.h, a.ctypes.data)); same(a)
    assert late.copied_bytes() == U * n * 4         # the frames there are, however long the stream may become
    r, k = dbls(U, CL, 64), ints(U, CL); c.ok(lib.mosaic_get_centroids(c.h, r.ctypes.data, k.ctypes.data)); same(r, k)
    s = dbls(U, n, 64); c.ok(lib.mosaic_get_summaries(c.h, s.ctypes.data)); same(s)
    c.ok(lib.mosaic_retrieve(c.h, 1, c.p, 1))
    ids, ni, sc = ints(2, 4), ints(2), dbls(2, CL)
    c.ok(lib.mosaic_get_selection(c.h, 1, ids.ctypes.data, ni.ctypes.data, sc.ctypes.data, None, 0, None)); same(ids, ni, sc)
    st = b.Stats(); c.ok(lib.mosaic_get_stats(c.h, C.byref(st))); assert st.sync_timeouts == 0 and st.frames_ingested == n
    # a later copy must not overwrite what the caller has changed since
    a[:] = 1; assert (a == 1).all() and late.late_copies_pending() == 0
c = Ctx(40, n_partitions=4, visual_dim=12)
fp, vr, vn, pr, pn = ints(40), dbls(4, 12), ints(4), dbls(U, 4, 64), ints(U, 4)
c.ok(lib.mosaic_get_partitions(c.h, *[x.ctypes.data for x in (fp, vr, vn, pr, pn)])); same(fp, vr, vn, pr, pn)
c.ok(lib.mosaic_retrieve(c.h, 2, c.p, 1))
pi, npi, ps = ints(2, 1), ints(2), dbls(2, 4)
c.ok(lib.mosaic_get_partition_selection(c.h, 2, pi.ctypes.data, npi.ctypes.data, ps.ctypes.data)); same(pi, npi, ps)
c = Ctx(40, maint_mode=b.MAINT_DEFERRED, init_clusters=4, buffer_max=3)
bf, bo = ints(U, 3), ints(U, 3)
c.ok(lib.mosaic_get_maintainer(c.h, None, None, None, None, None, bf.ctypes.data, bo.ctypes.data)); same(bf, bo)
print("OK")
"""


def test_observers_do_not_rely_on_asynchronous_copies(tmp_path):
    so = str(tmp_path / "late_copies.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "late_copies.c")])
    env = dict(os.environ, LD_PRELOAD=so, PYTHONPATH=os.path.dirname(HERE))
    p = subprocess.run([sys.executable, "-c", SCRIPT, so], env=env, capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(HERE))
    assert p.returncode == 0 and p.stdout.strip().endswith("OK"), p.stdout + p.stderr
