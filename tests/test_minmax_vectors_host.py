"""What the scan of the running estimates by position is launched with, without a GPU: vectors per thread by whether slabs are whole
vectors."""
from tests.launch_recorder import NAMES, run

BODY = r'''
def scan(layout, dt):
    st = L.mesa_update_running_params(P, dt, M.Layout(*layout), P, P, 0.9, 0, P, M.workspace_bytes(M.OP_UPDATE_RUNNING_PARAMS, *layout, dt), None)
    name, args, workgroups, threads, lds = kernels()[0]
    assert st == M.OK and name == "k_minmax_partial", (layout, st, name)
    return [int(args[args.index("Li") + 2:-1]), workgroups, lds]
'''


def test_vectors_per_thread():
    whole = [(25855, 16, 32), (619, 48, 256), (22583, 4, 64), (24, 4096, 96), (16, 8192, 64), (27276, 1, 196), (700, 8, 96), (7, 2048, 24), (3, 8192, 49), (25216, 6, 64), (200000, 12, 49), (2, 2048, 424), (1, 2048, 4088)]
    parts = [(8, 768, 49), (17001, 2, 20), (1, 2048, 441), (26330, 8, 49), (1358, 12, 49), (394, 3, 256), (600, 8, 96), (1, 4096, 49), (1, 768, 256), (1, 2048, 424), (1, 2048, 2024)]
    got = run(BODY + f"report([[(l, scan(l, dt)) for l in ls for dt in (M.F16, M.F32)] for ls in ({whole}, {parts})])", NAMES)
    assert all(how[0] == 4 and how[1] <= 1024 + 64 for _, how in got[0]), got[0]
    assert all(how[0] == 2 for _, how in got[1]), got[1]


def test_tables_of_extrema_per_workgroup():
    """Four where few groups' lanes meet, or slabs are long; one elsewhere (a minimum and a maximum of four bytes per group and table)."""
    four = [(25216, 6, 256), (128, 6, 38809), (619, 48, 256), (1117, 96, 128), (25855, 32, 32), (2560, 128, 96)]
    one = [(964, 128, 32), (991, 256, 16), (964, 256, 8), (1335, 192, 16), (700, 129, 256), (12000, 33, 64), (16, 8192, 64)]
    got = run(BODY + f"report([[(l, scan(l, M.F16)) for l in ls] for ls in ({four}, {one})])", NAMES)
    for tables, cases in zip((4, 1), got):
        assert all(lds == tables * 2 * 4 * l[1] for l, (_, _, lds) in cases), cases
