"""Which kernels the weight gradient takes, without a GPU."""
from tests.launch_recorder import NAMES, run


def routes(shapes):
    """[kernels, as (name, template arguments, workgroups, threads, LDS)] of (rows, K, N, type)"""
    return run(r'''
out = []
for Mr, K, N, dt in ''' + repr(list(shapes)) + r''':
    t = {"f16": M.F16, "bf16": M.BF16, "f32": M.F32}[dt]
    st = L.mesa_linear_dw_q(P, Mr, K, 1, P, P, P, N, t, P, P, P, M.workspace_bytes(M.OP_LINEAR_DW_Q, Mr, K, N, t), None)
    assert st == M.OK, (Mr, K, N, dt, st)
    out.append(kernels())
report(out)
''', NAMES)


def test_the_gpu_tests_of_the_tiles_reach_the_tiles():
    from tests.test_gpu_linear_dw_cut import EDGES, PLANS, RANGE, SPOILT
    cut = [(*s, "f32") for s in EDGES + RANGE + [SPOILT, (2500, 96, 72), (4099, 80, 136), (2300, 512, 512)]]
    got = routes(cut)
    assert all(k[0][0] == "k_dw_cut" for k in got), [(s, k[0][0]) for s, k in zip(cut, got)]
    assert {len(k) for k in got} == {1, 2}                  # one slice that finishes dW itself, and several
    tiles = [(Mr, K, N, dt) for Mr, K, N, *_ in PLANS for dt in ("f16", "bf16")]
    assert all(k[0][0] == "k_dw_f16" for k in routes(tiles))


def test_every_kernel_of_the_weight_gradient_is_reached():
    """by the shapes of the GPU tests, and by waves up to their lines."""
    shapes = [(Mr, K, N, dt) for Mr, K, N in ((50437, 768, 520), (50437, 400, 1000), (300, 8192, 8200), (300, 1008, 65536), (23451, 768, 1000), (4097, 768, 264), (505, 1344, 1088), (401408, 96, 288), (300, 640, 1032),
                                              (257, 640, 1024), (197, 512, 512), (100, 60, 72), (5000, 13, 9), (2081, 128, 128)) for dt in ("f16", "bf16", "f32")]
    got = routes(shapes)
    waves = {s: k[0][0] == "k_dw_waves" for s, k in zip(shapes, got)}
    assert all(waves[(*s, dt)] for s in ((257, 640, 1024), (197, 512, 512)) for dt in ("f16", "bf16", "f32"))
    assert not any(waves[(*s, dt)] for s in ((300, 640, 1032), (2081, 128, 128), (100, 60, 72)) for dt in ("f16", "bf16", "f32"))
    reached = {tuple(k[:2]) for ks in got for k in ks}
    there = {tuple(k) for k in run("report(all_kernels())", NAMES) if k[0].startswith("k_dw_")}
    assert there == reached, there ^ reached
