"""A launch of the Byzantine decoders that fails: the call returns APPROXIFER_ERR_LAUNCH and leaves every output as it was, whichever of its
launches it is (more than 128 classes: the votes' cells are cleared, the liars are located, the groups decoded)."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import launch_log

ENTRIES = ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"]

_RUN = r"""
import ctypes, json, sys
import numpy as np
sys.path.insert(0, sys.argv[3])
import launch_log
lib, log = launch_log.open_library(sys.argv[1], sys.argv[2])
hip = ctypes.CDLL("libamdhip64.so.7")
G, K, N, S, A, C = json.loads(sys.argv[4])
data = np.load(sys.argv[5])
def device(a):
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(max(a.nbytes, 256))) == 0
    assert hip.hipMemcpy(p, a.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(a.nbytes), 1) == 0
    return p
def back(p, like):
    a = np.empty_like(like)
    assert hip.hipMemcpy(a.ctypes.data_as(ctypes.c_void_p), p, ctypes.c_size_t(a.nbytes), 2) == 0
    return a
alpha, beta = (ctypes.c_double * K)(), (ctypes.c_double * N)()
lib.approxifer_chebyshev_nodes(K, N, alpha, beta)
host = (np.full((G, K, C), -3, np.float32), np.full((G, A), -7, np.int32), np.full(G, -9, np.int32))
preds, mask = device(data["preds"]), device(data["mask"])
seen = []
for entry in json.loads(sys.argv[6]):
    for with_workspace in (True, False):
        need = lib.approxifer_workspace_bytes(G, K, N, S, A, C) if with_workspace else 0
        assert not with_workspace or need >= 4 * G * (N + 1)
        ws = device(np.zeros(need, np.uint8)) if need else None
        fail, total = 0, 1
        while fail <= total:                               # the last time round no launch fails
            outs = [device(h) for h in host]
            log.launch_log_start(fail, 1)
            rc = getattr(lib, entry)(preds, mask, *outs, G, K, N, S, A, C, alpha, beta, 1, ws, need, None)
            total = len(log.launch_log().split())
            assert hip.hipDeviceSynchronize() == 0
            same = [bool(np.array_equal(back(p, h), h)) for p, h in zip(outs, host)]
            seen.append([entry, with_workspace, fail, total, rc, same])
            for p in outs: hip.hipFree(p)
            if rc == 0: break
            fail += 1
print(json.dumps(seen))
"""


@pytest.mark.gpu
@pytest.mark.parametrize("K,A,S,C", [(8, 2, 4, 300), (4, 1, 0, 1000)])
def test_outputs_stay_when_a_launch_fails(tmp_path, K, A, S, C):
    N, G = 2 * (K + A) + S, 3
    rng = np.random.default_rng(K)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[S:]] = 1
    np.savez(tmp_path / "in.npz", preds=rng.standard_normal((G, N, C)).astype(np.float32), mask=mask)
    r = subprocess.run([sys.executable, "-c", _RUN, launch_log.build_shim(str(tmp_path)), launch_log.library_path(),
                        os.path.dirname(os.path.abspath(__file__)), json.dumps([G, K, N, S, A, C]), str(tmp_path / "in.npz"),
                        json.dumps(ENTRIES)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    seen = json.loads(r.stdout)
    for entry, with_workspace, fail, total, rc, same in seen:
        if rc == 0:
            assert fail == total and not any(same), (entry, with_workspace)
        else:
            assert rc == -7 and all(same), (entry, with_workspace, fail, total, same)
    assert [s[4] for s in seen].count(0) == 2 * len(ENTRIES)
    assert max(s[3] for s in seen) == 3                      # clear, locate, decode
