"""Which kernels the attention products take, without a GPU."""
import re

from tests.launch_recorder import NAMES, run


def routes(shapes):
    """{(B, H, N, Dh, type): kernels of dA and dV, kernels of dQ and dK}, each as (name, template arguments, workgroups, threads, LDS)"""
    got = run(r'''
out = []
for B, H, N, Dh, dt in ''' + repr(list(shapes)) + r''':
    t = {"f16": M.F16, "bf16": M.BF16, "f32": M.F32}[dt]
    pair = []
    for st in (lambda: L.mesa_attn_av_bwd_q(P, P, B, H, N, Dh, P, P, P, P, P, P, P, t, None), lambda: L.mesa_attn_qk_bwd_q(P, P, B, H, N, Dh, P, P, P, P, P, 0.2, P, P, t, None)):
        assert st() == M.OK
        pair.append(kernels())
    out.append(pair)
report(out)
''', NAMES)
    return {s: [[tuple(k) for k in call] for call in g] for s, g in zip(shapes, got)}


def numbers(args):
    """the whole-number and truth arguments of a mangled template argument list"""
    return [int(x) for x in re.findall(r"L[a-z](\d+)E", args)]


def by_tiles(call):
    """groups of waves per workgroup of the column-tile kernel in a call, or None"""
    for name, args, _, threads, _ in call:
        if name == "k_attn_tn_cols":
            return threads // 256
    return None


def test_groups_of_waves_per_workgroup_of_the_column_tiles():
    want = {(1, 275, 200, 96, "f16"): 1, (1, 300, 130, 128, "bf16"): 1, (1, 200, 200, 96, "f16"): 2, (1, 300, 112, 128, "f16"): 1, (1, 256, 112, 96, "f16"): 1,
            (1, 300, 200, 64, "f16"): 2, (1, 300, 200, 32, "bf16"): 2, (1, 512, 112, 64, "f16"): 1, (1, 16, 4096, 64, "bf16"): 4, (1, 600, 200, 64, "f16"): 1}
    for shape, calls in routes(list(want)).items():
        assert [by_tiles(c) for c in calls] == [want[shape]] * 2, (shape, calls)
