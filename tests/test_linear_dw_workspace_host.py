"""The weight gradient's workspace, without a GPU: what the size query answers for a batch serves every smaller one too."""
from tests.launch_recorder import run


def test_a_workspace_sized_for_more_rows_serves_fewer():
    """A training loop sizes its workspace once, for the full batch, and its last batch is shorter: however the rows are
    cut into slices, no smaller number of them may need more."""
    bad = run(r'''
import random
rnd = random.Random(3)
bad, tried = [], 0
def call(rows, K, N, dt, n):
    st = L.mesa_linear_dw_q(P, rows, K, 1, P, P, P, N, dt, P, None, P, n, None)
    return st, len(launches())
shapes = [(384, 384, M.F16), (384, 1152, M.F16), (192, 768, M.F16), (192, 768, M.F32), (768, 3072, M.BF16), (96, 288, M.F16), (100, 60, M.F32), (3072, 768, M.BF16), (1536, 384, M.F16)]
for _ in range(60):
    shapes.append((16 * rnd.randint(1, 96), 8 * rnd.randint(1, 200), rnd.choice([M.F16, M.BF16, M.F32])))
for K, N, dt in shapes:
    for _ in range(12):
        full = int(2 ** rnd.uniform(5, 17))
        n = M.workspace_bytes(M.OP_LINEAR_DW_Q, full, K, N, dt)
        for _ in range(25):
            rows = rnd.randint(max(1, full // 2), full)
            tried += 1
            st, k = call(rows, K, N, dt, n)
            if st != M.OK or k not in (1, 2): bad.append((full, rows, K, N, dt, st, k))
assert tried > 20000, tried
for full, rows, K, N, dt in ((3200, 2961, 384, 384, M.F16), (1472, 1422, 384, 1152, M.F16), (3200, 2961, 192, 768, M.F16), (5824, 5488, 192, 768, M.F32)):
    st, k = call(rows, K, N, dt, M.workspace_bytes(M.OP_LINEAR_DW_Q, full, K, N, dt))
    if st != M.OK: bad.append((full, rows, K, N, dt, st, k))
report(bad)
''')
    assert not bad, bad[:10]


def test_a_workspace_that_is_too_small_is_refused():
    """Less than one slice for the small matrices, whose slices may be any number; less than eight ninths of the planned slices
    for the others, fewer than the plan of any larger matrix has."""
    got = run(r'''
out = []
for K, N, dt in ((384, 384, M.F16), (192, 768, M.F32), (1024, 256, M.BF16)):
    one = (N * K + N) * 4 + 16
    for n in (one, one - 16):
        st = L.mesa_linear_dw_q(P, 2961, K, 1, P, P, P, N, dt, P, None, P, n, None)
        out.append((st, len(launches())))
for K, N, dt, rows in ((768, 3072, M.F16, 50432), (96, 288, M.BF16, 401408)):
    n = M.workspace_bytes(M.OP_LINEAR_DW_Q, rows, K, N, dt)
    for m in (n, n * 4 // 5):
        st = L.mesa_linear_dw_q(P, rows, K, 1, P, P, P, N, dt, P, None, P, m, None)
        out.append((st, min(1, len(launches()))))
report(out)
''')
    for (st, k), (st0, k0) in zip(got[::2], got[1::2]):
        assert (st, k) == (0, 1) and (st0, k0) == (3, 0)
