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


KINDS = {"k_attn_da": "whole", "k_attn_tn": "whole", "k_attn_nn": "whole", "k_attn_da_cols": "tiles", "k_attn_tn_cols": "tiles", "k_attn_nn_rows": "tiles",
         "k_bmm_q": "general", "k_bmm_waves": "waves", "k_bmm_waves_two": "waves", "k_bmm_plain": "plain"}


def ways(shapes):
    """{shape: {product: way}}; a launch of two products stands for both"""
    out = {}
    for shape, calls in routes(shapes).items():
        w = {}
        for call, names in zip(calls, (("dA", "dV"), ("dQ", "dK"))):
            kinds = [KINDS[k[0]] for k in call]
            if len(kinds) == 1:
                kinds *= 2
            elif call[0][0] in ("k_attn_tn_cols", "k_attn_tn") or call[0][1].startswith("Lb1"):   # dV, whose first operand is coded, before dA
                kinds.reverse()
            w.update(zip(names, kinds))
        out[shape] = w
    return out


def test_short_heads_keep_a_workgroup_per_head():
    """dV and dK of very many heads of a few rows, and of fewer heads at a head size of 32."""
    want = {(1, 2048, 8, 128, "f16"): "whole", (1, 1536, 10, 128, "bf16"): "whole", (1, 1536, 12, 32, "f16"): "whole", (1, 571, 33, 32, "bf16"): "whole",
            (1, 650, 23, 96, "f16"): "whole", (1, 275, 71, 32, "f16"): "whole", (1, 28, 600, 32, "f16"): "tiles", (1, 200, 33, 96, "f16"): "general", (1, 300, 72, 64, "f16"): "general", (1, 132, 128, 96, "bf16"): "general", (1, 145, 128, 96, "bf16"): "tiles"}
    for shape, w in ways(list(want)).items():
        assert w["dV"] == w["dK"] == want[shape], (shape, w)


def test_heads_of_one_block_of_rows_keep_a_workgroup_each():
    """dV and dK of up to 32 rows, a wave per head, from a few hundred heads on; both products of dQ and dK by waves only up to 640 tiles in 16 bits."""
    want = {(1, 410, 16, 96, "f16"): "whole", (1, 450, 13, 96, "bf16"): "whole", (1, 582, 8, 128, "f16"): "whole", (1, 487, 32, 96, "f16"): "whole", (1, 733, 8, 64, "bf16"): "whole", (1, 340, 11, 64, "f16"): "whole",
            (1, 410, 33, 96, "f16"): "general", (1, 350, 8, 128, "f16"): "general", (1, 360, 8, 128, "f16"): "whole", (1, 641, 25, 32, "bf16"): "whole"}
    for shape, w in ways(list(want)).items():
        assert w["dK"] == w["dV"] == want[shape] and w["dQ"] != "waves", (shape, w)
    for shape, w in ways([(1, 640, 25, 32, "bf16"), (1, 320, 11, 64, "f16"), (1, 160, 44, 64, "f16")]).items():
        assert w["dQ"] == w["dK"] == "waves", (shape, w)


def test_da_of_medium_and_long_heads():
    """dA by tiles of aligned rows as soon as there are workgroups for it, of wide short heads and of unaligned rows up to 800 tokens whole."""
    want = {(1, 118, 224, 64, "f16"): "tiles", (1, 12, 760, 64, "bf16"): "tiles", (1, 12, 728, 128, "f16"): "tiles", (1, 250, 64, 64, "f16"): "general", (1, 403, 80, 96, "bf16"): "whole",
            (1, 822, 72, 96, "f16"): "whole", (1, 400, 88, 128, "f16"): "whole", (1, 27, 553, 64, "f16"): "whole", (1, 42, 463, 128, "f16"): "whole", (1, 28, 610, 32, "bf16"): "whole",
            (1, 192, 577, 64, "f16"): "tiles", (1, 192, 420, 64, "f16"): "whole", (1, 60, 919, 64, "f16"): "tiles", (1, 16, 4096, 64, "bf16"): "tiles", (1, 768, 197, 64, "f16"): "whole",
            (1, 403, 96, 96, "f16"): "tiles", (1, 403, 72, 64, "f16"): "tiles", (1, 11, 511, 64, "f16"): "general", (1, 38, 687, 64, "bf16"): "tiles", (1, 38, 687, 128, "bf16"): "whole", (1, 18, 733, 64, "bf16"): "whole",
            (1, 9, 544, 64, "f16"): "general", (1, 44, 524, 64, "f16"): "whole", (1, 24, 765, 64, "f16"): "tiles", (1, 41, 655, 96, "f16"): "tiles"}
    for shape, w in ways(list(want)).items():
        assert w["dA"] == want[shape], (shape, w)


def test_dq_of_many_short_and_of_long_heads():
    """dQ whole of many unaligned short heads, by tiles of long ones only once there are workgroups for it."""
    want = {(1, 949, 125, 32, "f16"): "whole", (1, 750, 118, 32, "f16"): "whole", (1, 1550, 80, 32, "bf16"): "tiles", (1, 516, 97, 128, "f16"): "whole", (1, 16, 888, 96, "bf16"): "general",
            (1, 11, 1126, 128, "bf16"): "general", (1, 14, 1426, 64, "bf16"): "general", (1, 19, 1356, 64, "f16"): "general", (1, 16, 4096, 64, "bf16"): "tiles", (1, 60, 919, 64, "f16"): "tiles",
            (1, 192, 301, 96, "f16"): "tiles", (1, 768, 197, 64, "f16"): "whole", (1, 64, 601, 32, "f16"): "tiles", (1, 24, 919, 96, "f16"): "tiles", (1, 55, 512, 64, "f16"): "tiles", (1, 15, 1168, 128, "bf16"): "tiles", (1, 526, 144, 128, "f16"): "tiles"}
    for shape, w in ways(list(want)).items():
        assert w["dQ"] == want[shape], (shape, w)


def test_few_heads_by_waves_only_where_that_is_faster():
    """Both products in one launch, one alone, and neither; in binary32 with four waves by how the tiles compare with the general kernel's."""
    want = {(1, 6, 197, 64, "f32"): ("waves", "waves", "waves"), (1, 490, 53, 64, "f32"): ("general", "general", "general"), (1, 391, 60, 64, "f32"): ("general", "general", "general"),
            (1, 290, 39, 64, "f32"): ("general", "waves", "waves"), (1, 1653, 20, 32, "f32"): ("waves", "waves", "waves"), (1, 464, 24, 128, "f32"): ("waves", "general", "general"),
            (1, 10, 1248, 64, "f32"): ("general", "general", "waves"), (1, 12, 783, 64, "f32"): ("general", "waves", "waves"), (1, 128, 120, 64, "f32"): ("general", "general", "general"),
            (1, 261, 92, 16, "f32"): ("general", "waves", "waves"), (1, 65, 112, 96, "f32"): ("general", "waves", "waves"), (1, 696, 43, 32, "f32"): ("general", "general", "waves"),
            (1, 78, 65, 64, "f16"): ("whole", "waves", "waves"), (1, 156, 44, 64, "f16"): ("whole", "general", "waves"), (1, 4, 2048, 64, "f16"): ("tiles", "waves", "waves"),
            (1, 3, 436, 64, "bf16"): ("waves", "waves", "waves"), (1, 1, 8192, 64, "bf16"): ("tiles", "waves", "waves"),
            (1, 3, 8192, 32, "f32"): ("general", "waves", "waves"), (1, 6, 2047, 64, "f32"): ("general", "waves", "waves"), (1, 272, 27, 80, "f16"): ("waves", "general", "general")}
    for shape, w in ways(list(want)).items():
        assert (w["dA"], w["dV"], w["dK"]) == want[shape] and (w["dQ"] == "waves") == (w["dK"] == "waves"), (shape, w)


def test_dv_goes_first_beside_a_da_as_large_as_the_memory_side_cache():
    first = {(1, 7, 4096, 64, "bf16"): "dV", (1, 8, 4096, 64, "bf16"): "dV", (32, 12, 577, 64, "f16"): "dV", (256, 12, 250, 64, "f16"): "dV", (8, 12, 1024, 64, "f16"): "dA",
             (1, 6, 4096, 64, "bf16"): "dA", (1, 16, 4096, 64, "f32"): "dA",
             (1, 1831, 256, 96, "f16"): "dA", (12, 1221, 128, 64, "bf16"): "dA", (1, 5182, 224, 64, "f16"): "dV", (1, 1447, 288, 32, "f16"): "dV",   # of up to 256 elements not if dA leaves non-temporally
             (1, 2219, 352, 64, "f16"): "dA", (1, 549, 640, 64, "bf16"): "dV", (1, 1221, 640, 64, "bf16"): "dA", (1, 128, 4096, 64, "f16"): "dV", (1, 3840, 250, 64, "f16"): "dV"}   # nor of more than 600000
    for shape, (av, _) in routes(list(first)).items():
        got = "dV" if av[0][0] == "k_attn_tn_cols" or av[0][1].startswith("Lb1") else "dA"
        assert len(av) == 2 and got == first[shape], (shape, av)


# for `also`: an argument of a launch that says how its kernel goes about the memory: k_attn_da_cols' eighth (stores past the caches), k_attn_nn_rows' seventh (tiles start at
# different columns); -1 for other kernels
HOW = r'''
static int how_[64];
void launched(int at, const void *f, void **args)
{
    how_[at] = -1;
    for (int k = 0; k < known_n; ++k) {
        if (known[k].f != f) continue;
        if (strstr(known[k].name, "14k_attn_da_cols")) how_[at] = *(int *)args[7];
        if (strstr(known[k].name, "14k_attn_nn_rows")) how_[at] = *(int *)args[6];
    }
}
int recorded_how(int i) { return how_[i]; }
'''


def how(call, shapes):
    got = run(r'''
out = []
for b, N, Dh in ''' + repr(list(shapes)) + r''':
    assert (''' + call + r''') == M.OK
    out.append(max(rec.recorded_how(i) for i in range(len(launches()))))
report(out)
''', NAMES + HOW)
    return dict(zip(shapes, got))


def test_da_by_tiles_leaves_past_the_caches_by_its_real_size():
    """Rows of a multiple of 128 elements from 170 MB on (of 128 from 100), whatever part of their last tile exists; rows on half lines from 256 elements on, but not those of more
    than 448 in heads of up to 64 that take about half of the memory-side cache; never rows that start elsewhere."""
    want = {(3051, 128, 64): 0, (3052, 128, 64): 1, (576, 384, 64): 0, (577, 384, 128): 1, (1296, 256, 64): 0, (1298, 256, 32): 1, (81, 1024, 64): 0, (82, 1024, 64): 1,
            (5, 4096, 64): 0, (6, 4096, 64): 1, (64, 1152, 64): 0, (65, 1152, 64): 1, (2170, 96, 64): 0, (10851, 96, 64): 0, (399, 224, 64): 0, (90, 288, 64): 1, (562, 320, 32): 1, (324, 448, 64): 1,
            (25, 480, 64): 1, (227, 480, 64): 1, (229, 480, 64): 0, (336, 480, 64): 0, (337, 480, 64): 1, (131, 704, 96): 1, (166, 576, 128): 1, (20, 2016, 64): 0, (23, 2016, 64): 1,
            (51, 656, 64): 0, (192, 577, 64): 0}
    got = how("L.mesa_attn_av_bwd_q(P, P, 1, b, N, Dh, P, P, P, P, P, P, P, M.BF16, None)", want)
    assert got == want, {s: g for s, g in got.items() if want[s] != g}


def test_dq_by_tiles_starts_at_different_columns_where_rows_meet_on_the_same_channels():
    """Rows of a multiple of 1024 elements from 2048 on, of a dS of up to 750 MB."""
    want = {(16, 4096, 64): 1, (22, 4096, 64): 1, (23, 4096, 64): 0, (128, 4096, 64): 0, (36, 2048, 32): 1, (89, 2048, 64): 1, (90, 2048, 64): 0, (16, 3072, 64): 1, (9, 4096, 128): 1, (10, 5120, 32): 1,
            (67, 1024, 64): 0, (34, 2112, 64): 0, (17, 1536, 96): 0, (9, 4160, 64): 0, (114, 512, 64): 0, (150, 320, 64): 0, (64, 601, 32): 0}
    got = how("L.mesa_attn_qk_bwd_q(P, P, 1, b, N, Dh, P, P, P, P, P, 0.2, P, P, M.BF16, None)", want)
    assert got == want, {s: g for s, g in got.items() if want[s] != g}


def test_the_gpu_tests_reach_every_kernel_of_the_products():
    """and no kernel is there that no call reaches."""
    from tests.test_gpu_attention_kernels import SIXTEEN, WIDE
    shapes = [(*s, t) for s in SIXTEEN for t in ("f16", "bf16")] + [(*s, "f32") for s in WIDE]
    reached = {k[:2] for calls in routes(shapes).values() for call in calls for k in call}
    there = {tuple(k) for k in run("report(all_kernels())", NAMES) if k[0] in KINDS}
    assert there and there == reached, there ^ reached


def test_heads_over_the_range_of_binary32_go_to_the_general_kernel():
    w = ways([(1, 22, 600, 64, "f32")])[(1, 22, 600, 64, "f32")]
    assert set(w.values()) == {"general"}, w
