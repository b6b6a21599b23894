"""The library's host side on a recording stand-in of the HIP runtime (host_stub.py):
what it launches, refuses and sizes, at sizes and failures that need no GPU."""
import host_stub


def test_appended_rows_beyond_32_bits(tmp_path):
    """Steps that append batch x n_new rows of `hidden` columns, 2^31 and 2^32 values of
    them among the sizes: the launch that writes the rows as fragment planes has eight columns
    a thread, no more threads than a grid holds, and none missing."""
    host_stub.run('''
for fuse in (0, 5):
    m = h.Model(h.config(4096, 32, 12288, vocab=4096, fuse=fuse))
    for batch, n_new in ((1, 1), (3, 7), (64, 8191), (64, 8192), (64, 16448)):
        st = m.step(batch, 17000, n_new, 1 << 40)
        assert st == 0, (batch, n_new, st)
        grids = [r for r in h.log() if r[0] == "launch" and "sum_parts_planes" in r[1]]
        assert len(grids) == 1
        threads = int(grids[0][2]) * int(grids[0][5])
        assert batch * n_new * 4096 // 8 <= threads < 2**32, (fuse, batch, n_new, threads)
        assert grids[0][3:5] == ["1", "1"]
''', tmp_path)
