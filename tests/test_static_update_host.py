"""The update on the library's own array, without a GPU: every layout of up to 4096 groups is launched, on no more workgroups than
the array has room for."""
from tests.launch_recorder import ONE_DEVICE, run


def test_every_layout_of_up_to_4096_groups_fits_the_array():
    bad = run(r'''
import random
rnd = random.Random(5)
bad = []
room = L.mesa_static_scratch_bytes()
def call(layout, dt=M.F16):
    st = L.mesa_update_running_params_static(P, dt, M.Layout(*layout), P, P, 0.9, 0, None)
    k = launches()
    if st != M.OK or len(k) not in (1, 2): return bad.append((layout, st, k))
    by_group = k[0][3] == 1024
    workgroups = k[0][1] if by_group else k[0][0]          # whose extrema of `groups` groups go to the array
    if len(k) == 2 and workgroups * 2 * layout[1] * 4 > room: bad.append((layout, "room", k))
for layout in ((12, 4096, 64), (37, 1024, 49), (37, 768, 256), (84, 1536, 64), (1321, 128, 49), (209, 768, 96), (26, 2048, 96), (1589, 384, 20),
               (54, 3072, 64), (2662, 128, 49), (983, 768, 20), (1, 1024, 9001), (1, 4096, 1), (4096, 4096, 1)):
    call(layout)
for groups in range(1, 4097):
    for size in (1 << 12, 1 << 20, 1 << 23, (1 << 24) - 4096, (1 << 24) + 4096, 1 << 26):
        inner = rnd.choice((1, 8, 20, 49, 64, 96, 256, rnd.randint(1, 3000)))
        call((max(1, size // (groups * inner)), groups, inner), rnd.choice((M.F16, M.F32)))
for _ in range(20000):
    groups = int(2 ** rnd.uniform(0, 12))
    inner = int(2 ** rnd.uniform(0, 12))
    call((max(1, int(2 ** rnd.uniform(10, 28)) // (groups * inner)), groups, inner))
report([len(bad), bad[:8]])
''', ONE_DEVICE)
    assert bad[0] == 0, bad
