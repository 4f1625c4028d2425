"""Codec calls in which a wave takes several narrow rows, against the same rows in
calls small enough that it takes one.

Both forms use the same operations in the same order, so codes, scales, row sums
and reconstructions must agree bit for bit (the small calls are pinned against the
oracle in test_gpu_codec.py); guard bytes around every output show stray writes.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 64  # elements on either side of an output, keeps 16-byte alignment


def guarded(n, dtype):
    buf = torch.full((n + 2 * GUARD,), 77, dtype=dtype, device="cuda")
    return buf, buf[GUARD:GUARD + n]


def make(rows, cols, block, ld, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((rows, ld), generator=g, device="cuda")
    x[:, ::37] *= 30.0
    x[rows // 3] = 0.0
    x[rows // 2] *= 2.0 ** -70
    u = {"x": x.to(torch.bfloat16)[:, :cols], "rows": rows, "cols": cols, "ld": ld}
    for k, n, t in (("codes", rows * cols, torch.uint8), ("xhat", rows * cols, torch.bfloat16),
                    ("ss_x", rows, torch.float32), ("ss_err", rows, torch.float32),
                    ("scales", rows * (cols // block) if block else 0, torch.float32)):
        u[k + "_buf"], u[k] = guarded(n, t)
    return u


def desc(hl, u, r0, r1, block, stats):
    c, nb = u["cols"], u["cols"] // block if block else 0
    sl = lambda k, w: u[k][r0 * w:r1 * w].view(r1 - r0, w)  # noqa: E731
    return hl.unit_desc(x=u["x"][r0:r1], codes=sl("codes", c), xhat=sl("xhat", c),
                        scales=sl("scales", nb) if block else None,
                        row_ss_x=u["ss_x"][r0:r1] if stats else None,
                        row_ss_err=u["ss_err"][r0:r1] if stats else None, rows=r1 - r0, cols=c,
                        ld=u["ld"])


OUT = ("codes", "scales", "xhat", "ss_x", "ss_err")


@pytest.mark.parametrize("code,block,widths", [
    (0, 32, (32, 96, 256, 288, 512, 544, 1024)),
    (0, 256, (256, 512, 768, 1024)),
    (1, 64, (64, 192, 320, 896)),
    (1, 128, (128, 256, 512, 640, 1024)),
    (2, 0, (8, 248, 256, 264, 512, 520, 1000, 1024, 1032)),
], ids=["int8-32", "int8-256", "e4m3fn-64", "e4m3fn-128", "cast"])
@pytest.mark.parametrize("stats", [True, False], ids=["sums", "plain"])
def test_groups_match_single_rows(hl, code, block, widths, stats):
    # row counts leave a part of a group at the end of units; one stride is padded
    shapes = [(2333 - 16 * i + i, w, w + (24 if i == 1 else 0)) for i, w in enumerate(widths)]
    shapes.append((8192, widths[0], widths[0]))  # the call has 8192 rows and more
    many = [make(r, c, block, ld, 10 * i + code) for i, (r, c, ld) in enumerate(shapes)]
    few = [make(r, c, block, ld, 10 * i + code) for i, (r, c, ld) in enumerate(shapes)]
    units = [desc(hl, u, 0, u["rows"], block, stats) for u in many]
    hl.hilore_compress(units, code, block)
    hl.hilore_decompress(units, code, block)
    for u in few:
        for r0 in range(0, u["rows"], 4096):  # slices below the limit, 16-byte aligned
            part = [desc(hl, u, r0, min(u["rows"], r0 + 4096), block, stats)]
            hl.hilore_compress(part, code, block)
            hl.hilore_decompress(part, code, block)
    for u, v in zip(many, few):
        for k in OUT:
            a, b = (t[k + "_buf"].view(torch.uint8) for t in (u, v))
            assert torch.equal(a, b), (u["rows"], u["cols"], k)
            if k not in ("ss_x", "ss_err") or stats:
                w = u[k + "_buf"]
                assert bool((w[:GUARD] == 77).all()) and bool((w[-GUARD:] == 77).all())


@pytest.mark.parametrize("code,block", [(0, 64), (1, 128), (2, 0)], ids=["int8", "e4m3fn", "cast"])
@pytest.mark.parametrize("shapes", [
    [(5001, 896), (4099, 640)],            # every unit two rows per wave,
    [(4097, 512), (4098, 384)],            # four,
    [(8193, 128), (1, 256)],               # eight
    [(4097, 128), (2, 2560), (4099, 1024), (3, 2048), (1003, 1152), (7, 2688), (5, 256),
     (9001, 896), (1, 384)],               # all sizes and single rows, two row mappings
], ids=["two", "four", "eight", "mixed"])
def test_launches_of_one_size_and_of_several(hl, code, block, shapes):
    many = [make(r, c, block, c, 10 * i + code) for i, (r, c) in enumerate(shapes)]
    few = [make(r, c, block, c, 10 * i + code) for i, (r, c) in enumerate(shapes)]
    units = [desc(hl, u, 0, u["rows"], block, True) for u in many]
    hl.hilore_compress(units, code, block)
    hl.hilore_decompress(units, code, block)
    for u in few:
        for r0 in range(0, u["rows"], 4096):
            part = [desc(hl, u, r0, min(u["rows"], r0 + 4096), block, True)]
            hl.hilore_compress(part, code, block)
            hl.hilore_decompress(part, code, block)
    for u, v in zip(many, few):
        for k in OUT:
            a, b = (t[k + "_buf"].view(torch.uint8) for t in (u, v))
            assert torch.equal(a, b), (u["rows"], u["cols"], k)
            w = u[k + "_buf"]
            assert bool((w[:GUARD] == 77).all()) and bool((w[-GUARD:] == 77).all())


def test_cast_rows_of_any_length_share_a_launch(hl):
    """Rows of the literal cast may end inside an 8-column piece; such a unit keeps one row
    per wave in a launch whose other units are grouped."""
    shapes = [(8200, 128), (333, 13), (1001, 896), (7, 2001), (65, 1023), (4099, 264)]
    many = [make(r, c, 0, -(-c // 8) * 8, 10 * i) for i, (r, c) in enumerate(shapes)]
    few = [make(r, c, 0, -(-c // 8) * 8, 10 * i) for i, (r, c) in enumerate(shapes)]
    units = [desc(hl, u, 0, u["rows"], 0, True) for u in many]
    hl.hilore_compress(units, 2, 0)
    hl.hilore_decompress(units, 2, 0)
    for u in few:
        for r0 in range(0, u["rows"], 4096):
            part = [desc(hl, u, r0, min(u["rows"], r0 + 4096), 0, True)]
            hl.hilore_compress(part, 2, 0)
            hl.hilore_decompress(part, 2, 0)
    for u, v in zip(many, few):
        for k in OUT:
            a, b = (t[k + "_buf"].view(torch.uint8) for t in (u, v))
            assert torch.equal(a, b), (u["rows"], u["cols"], k)
            w = u[k + "_buf"]
            assert bool((w[:GUARD] == 77).all()) and bool((w[-GUARD:] == 77).all())
