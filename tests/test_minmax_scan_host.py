"""Which scan the running estimates take, without a GPU: by group is for slabs that its vectors fit and for groups that fill a
workgroup."""
from tests.launch_recorder import run


def test_scan_by_group_only_where_it_pays():
    got = run(r'''
def scan(layout, dt=M.F16, scale_only=False):
    n = M.workspace_bytes(M.OP_UPDATE_RUNNING_PARAMS, *layout, dt)
    st = L.mesa_update_running_params(P, dt, M.Layout(*layout), P, P, 0.9, 0, P, n, None)
    k = launches()
    assert st == M.OK and len(k) in (1, 2), (layout, st, k)
    assert (len(k) == 1) == (k[0][3] == 1024 and k[0][1] == 1), (layout, k)
    return "one" if len(k) == 1 else "pieces" if k[0][3] == 1024 else "position"
# strided elements, slabs shorter than a vector, workgroups with nothing to do, and large tensors of few groups
slow = [(32768, 768, 1), (25216, 384, 1), (25216, 64, 1), (32768, 16, 1), (16384, 64, 2), (4096, 96, 8), (4096, 768, 8), (4096, 8192, 4), (2048, 384, 7),
        (4096, 2048, 6), (1, 8192, 1), (4, 8192, 1), (1, 8192, 64), (1, 8192, 100), (1, 4096, 64), (16, 4096, 128), (11184, 2, 1500), (82241, 3, 68),
        (15420, 8, 68), (64527, 2, 65), (8196, 2, 2047), (100000, 12, 20), (8192, 3, 2401)]
fast = [(394, 3, 64), (64, 8, 441), (394, 192, 1), (394, 384, 1), (1024, 16, 20), (16, 512, 49), (128, 768, 196), (8, 768, 4096), (100, 8192, 100), (512, 384, 64),
        (16, 2048, 65), (32768, 1, 1), (1, 1, 1), (1023, 2, 1), (1000, 8192, 65)]
pieces = [(725, 8, 341), (1919, 32, 441), (50000, 3, 341), (200, 768, 196)]
report([[(l, scan(l)) for l in ls] for ls in (slow, fast, pieces)])
''')
    for want, cases in zip(("position", "one", "pieces"), got):
        assert all(how == want for _, how in cases), (want, [c for c in cases if c[1] != want])
