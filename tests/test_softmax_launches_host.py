"""Softmax at the largest numbers of rows, without a GPU: every B * H * rows below 2^31 is a launch that the hardware can
be given, whatever the row length and the type (the tensors would not all fit a card, their calls are still accepted)."""
from tests.launch_recorder import run


def test_softmax_launches_fit_at_any_number_of_rows():
    bad = run(r'''
P2, P3, bad, tried = 0x20000, 0x30000, [], 0
ws = 1 << 40
for cols in (1, 8, 49, 197, 256, 257, 264, 384, 513, 520, 577, 769, 1000, 1023, 1025, 1032, 1500, 1999, 2047, 2048, 2050, 2056, 3080, 4095, 4096, 4104, 9000):
    for H in (1, 12, 2000):
        for lg in (20, 24, 26, 27, 28, 29, 30, 31):
            rows = ((1 << lg) - 1) // H
            for dt in (M.F32, M.F16, M.BF16):
                st = L.mesa_softmax_bwd_q(P, 1, H, rows, cols, P, P, P2, P3, dt, None)
                k = launches()
                tried += 1
                if st != M.OK or len(k) != 1: bad.append(("bwd", cols, H, rows, dt, st, k))
                if rows * cols < 1 << 30 and H * rows * cols < 1 << 50:
                    st = L.mesa_softmax_fwd_q(P, 1, H, rows, cols, P, P, 0.9, P2, P3, 1, 0, 0, P, ws, dt, None)
                    k = launches()
                    if st != M.OK: bad.append(("fwd", cols, H, rows, dt, st, k))
report(bad)
''')
    assert not bad, (len(bad), bad[:6])
