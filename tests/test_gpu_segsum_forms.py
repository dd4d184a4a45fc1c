"""Seg-Sum's forms: rows whose width or start is no multiple of a 16-byte
vector, updates whose table rows load early or late, and segments cut into any
number of pieces."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gpu_helpers as H  # noqa: E402
import oracle  # noqa: E402
from paper_1810_10045_amd import synth  # noqa: E402

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def lz():
    from paper_1810_10045_amd import lmzipf
    return lmzipf


# Widths around one vector (4 fp32, 8 bf16 columns), around a fix-up tile (256)
# and a walk tile (1024) with less than a vector in the last one (1025..1027
# fp32, ..1031 bf16), past the one-launch form (4097), and the first column.
WIDTHS = [("f32", D, o) for D, o in ((3, 0), (4, 1), (5, 0), (7, 0), (255, 0), (257, 1), (650, 0),
                                     (1022, 1), (1024, 3), (1025, 0), (1027, 0), (2049, 0),
                                     (4097, 0))] + \
         [("bf16", D, o) for D, o in ((7, 0), (8, 1), (9, 0), (300, 0), (517, 1), (1023, 0),
                                      (1028, 0), (1031, 0), (2048, 4), (4095, 0))]


@pytest.mark.parametrize("gdt,D,first", WIDTHS, ids=[f"{g}-D{d}+{o}" for g, d, o in WIDTHS])
def test_segsum_any_width(lz, gdt, D, first):
    """The sums against the oracle (rows of one token exact); into table rows,
    and with SGD and Adam, bit for bit what lm_segsum and then the call of its
    own give; columns outside the table's D untouched."""
    K, V = 5000, 700
    print(f"segsum {gdt} D={D} first column {first}", flush=True)
    ids = synth.zipf_ids_permuted(K, V, 1.1, 300 + D, 5, np.int32)
    wide = torch.from_numpy(synth.normal_rows(K, D + 5, 301 + D)).to(DEV)
    wide = wide.to(torch.bfloat16) if gdt == "bf16" else wide
    grad = wide[:, first:first + D]
    r = lz.unique(torch.from_numpy(ids).to(DEV), V)
    seg = (grad, r.perm, r.inverse, r.offsets, r.num_unique)
    sums = lz.segsum(*seg, dev_err=r.dev_err)
    base = torch.from_numpy(synth.normal_rows(V, D + 5, 302 + D, 0.02)).to(DEV)

    def table():
        t = base.clone()
        return t, t[:, first:first + D]

    whole = {}
    for how in ("rows", "sgd", "adam"):
        t1, a = table()
        t2, b = table()
        if how == "rows":
            lz.segsum_rows(*seg, r.uniq, a, dev_err=r.dev_err)
            lz.fill_values(sums, r.uniq, r.num_unique, b, mode="scatter", dev_err=r.dev_err)
        elif how == "sgd":
            lz.segsum_sgd(*seg, r.uniq, a, 0.1, dev_err=r.dev_err)
            lz.sparse_apply(b, r.uniq, r.num_unique, sums, "sgd", lr=0.1, dev_err=r.dev_err)
        else:
            m1, v1 = table()[1].abs(), table()[1].square()
            m1, v1 = (torch.empty_like(t1)[:, first:first + D].copy_(x) for x in (m1, v1))
            m2, v2 = (torch.empty_like(t1)[:, first:first + D].copy_(x) for x in (m1, v1))
            lz.segsum_adam(*seg, r.uniq, a, m1, v1, step=3, dev_err=r.dev_err)
            lz.sparse_apply(b, r.uniq, r.num_unique, sums, "adam", lr=1e-3, step=3, m=m2, v=v2,
                            dev_err=r.dev_err)
            assert torch.equal(m1, m2) and torch.equal(v1, v2), "moments differ"
        assert torch.equal(t1, t2), f"{how}: not lm_segsum and then the call of its own"
        outside = torch.ones(D + 5, dtype=torch.bool)
        outside[first:first + D] = False
        assert torch.equal(t1[:, outside], base[:, outside]), f"{how}: wrote outside its columns"
        whole[how] = t1
    torch.cuda.synchronize()
    lz.check(r.dev_err)
    o = H.assert_unique_matches(r, ids, V, oracle)
    U = len(o[0])
    host = (np.ascontiguousarray(grad.contiguous().view(torch.int16).cpu().numpy().view(np.uint16))
            if gdt == "bf16" else np.ascontiguousarray(grad.cpu().numpy()))
    ref = oracle.segsum(host, o[3], U)
    got = sums[:U].double().cpu().numpy()
    H.check_rows(got, ref, H.sum_of_squares(host, o[3], U, oracle), gdt)
    H.assert_single_rows_exact(got, ref, o[1])


@pytest.mark.parametrize("D,first", [(63, 0), (64, 0), (65, 1), (66, 1), (127, 0), (129, 0), (255, 0),
                                     (256, 0), (257, 0), (250, 0), (251, 0)])
def test_segsum_bf16_rows_between_words(lz, D, first):
    """bf16 rows of odd width, stride or start: up to 256 columns a column per
    lane (1, 2 and 4 for each lane), from there on vectors."""
    test_segsum_any_width(lz, "bf16", D, first)


@pytest.mark.parametrize("K,V,D,gdt", [(6400, 199, 1024, "f32"), (6400, 200, 512, "f32"),
                                       (6400, 201, 650, "f32"), (300_000, 200_000, 64, "f32"),
                                       (9000, 8000, 520, "bf16"), (5000, 1, 300, "f32")])
def test_updates_on_either_side_of_the_early_rule(lz, K, V, D, gdt):
    """SGD's table rows load with the gradient rows below 32 tokens per type
    (fp32, chunks below 512 rows), else, and for Adam, after each segment: the
    tables are those of lm_segsum and then lm_sparse_apply, bit for bit."""
    print(f"update K={K} V={V} D={D} {gdt}", flush=True)
    ids = torch.from_numpy(synth.zipf_ids(K, V, 1.0, 400 + K, np.int64)).to(DEV)
    grad = torch.from_numpy(synth.normal_rows(K, D, 401 + K)).to(DEV)
    grad = grad.to(torch.bfloat16) if gdt == "bf16" else grad
    r = lz.unique(ids, V)
    seg = (grad, r.perm, r.inverse, r.offsets, r.num_unique)
    sums = lz.segsum(*seg, dev_err=r.dev_err)
    p = torch.from_numpy(synth.normal_rows(V, D, 402, 0.02)).to(DEV)
    m, v = p.clone(), p.square()
    a, b = p.clone(), p.clone()
    lz.segsum_sgd(*seg, r.uniq, a, 0.1, dev_err=r.dev_err)
    lz.sparse_apply(b, r.uniq, r.num_unique, sums, "sgd", lr=0.1, dev_err=r.dev_err)
    assert torch.equal(a, b)
    t1, t2 = ([x.clone() for x in (p, m, v)] for _ in range(2))
    lz.segsum_adam(*seg, r.uniq, *t1, step=2, weight_decay=0.01, dev_err=r.dev_err)
    lz.sparse_apply(t2[0], r.uniq, r.num_unique, sums, "adam", lr=1e-3, step=2, weight_decay=0.01,
                    m=t2[1], v=t2[2], dev_err=r.dev_err)
    assert all(torch.equal(x, y) for x, y in zip(t1, t2))
    lz.check(r.dev_err)


@pytest.mark.parametrize("length", [1, 7, 8, 16, 17, 31, 100, 255, 256, 257, 300, 1500, 6000])
@pytest.mark.parametrize("D,gdt", [(512, "f32"), (1500, "f32"), (1100, "bf16")])
def test_segments_of_one_length(lz, length, D, gdt):
    """Types of `length` tokens each, over a list with room for far more types:
    lengths around the shortest cut segment, one and several pieces, and the 16
    further pieces from which a fix-up workgroup sums them; repeated calls on
    one workspace agree, and so do the two launch forms within the tolerance."""
    K, V = 6000, 100_000
    print(f"segments of {length} D={D} {gdt}", flush=True)
    base = np.repeat(np.arange((K + length - 1) // length) * 16 + 3, length)[:K].astype(np.int32)
    ids = np.random.Generator(np.random.PCG64(length)).permutation(base)
    g = torch.from_numpy(synth.normal_rows(K, D, 500 + length)).to(DEV)
    g = g.to(torch.bfloat16) if gdt == "bf16" else g
    ws = lz.Workspace(DEV)
    r = lz.unique(torch.from_numpy(ids).to(DEV), V, ws=ws)
    seg = (g, r.perm, r.inverse, r.offsets, r.num_unique)
    one = [lz.segsum(*seg, dev_err=r.dev_err, ws=ws) for _ in range(3)]
    assert lz.segsum_two_launches(True) is False
    try:
        two = lz.segsum(*seg, dev_err=r.dev_err, ws=ws)
    finally:
        assert lz.segsum_two_launches(False) is True
    torch.cuda.synchronize()
    lz.check(r.dev_err)
    o = H.assert_unique_matches(r, ids, V, oracle)
    U = len(o[0])
    assert all(torch.equal(one[0][:U], x[:U]) for x in one[1:]), "not the same bits every time"
    host = (g.view(torch.int16).cpu().numpy().view(np.uint16) if gdt == "bf16" else g.cpu().numpy())
    ref = oracle.segsum(host, o[3], U)
    for got in (one[0], two):
        got = got[:U].double().cpu().numpy()
        H.check_rows(got, ref, H.sum_of_squares(host, o[3], U, oracle), gdt)
        H.assert_single_rows_exact(got, ref, o[1])


@pytest.mark.parametrize("K,V,D,gdt", [(16_385, 98, 200, "f32"), (21_386, 2865, 357, "f32"),
                                       (60_000, 500, 358, "f32"), (40_000, 2000, 300, "bf16")])
def test_sums_where_chunks_are_made_to_fill_the_device(lz, K, V, D, gdt):
    """Chunk counts raised to a number of waves: whole and part vectors, chunks
    down to 16 rows, heads and short cut segments. Rows of small whole numbers,
    whose sums are exact in fp32 in any order."""
    print(f"filled K={K} V={V} D={D} {gdt}", flush=True)
    ids = torch.from_numpy(synth.zipf_ids(K, V, 1.1, 700 + K, np.int32)).to(DEV)
    grad = torch.from_numpy(np.random.Generator(np.random.PCG64(K)).integers(-8, 9, (K, D))).to(DEV)
    want = torch.zeros((V, D), dtype=torch.int64, device=DEV).index_add_(0, ids.long(), grad)
    grad = grad.to(torch.bfloat16 if gdt == "bf16" else torch.float32)
    r = lz.unique(ids, V)
    out = lz.segsum(grad, r.perm, r.inverse, r.offsets, r.num_unique, dev_err=r.dev_err)
    lz.check(r.dev_err)
    U = int(r.num_unique.item())
    assert torch.equal(out[:U].double(), want[r.uniq[:U].long()].double())


@pytest.mark.parametrize("length", [1, 9, 40, 300, 1500])
@pytest.mark.parametrize("D,gdt", [(5, "f32"), (517, "f32"), (1022, "f32"), (9, "bf16"), (1101, "bf16")])
def test_pieces_of_rows_that_are_no_whole_vectors(lz, length, D, gdt):
    """Cut segments of `length` tokens whose partial rows start at the alignment
    of a float: a few pieces, the sixteenth, and heads; written, and applied by
    SGD and Adam. Rows of small whole numbers, whose sums are exact in fp32."""
    K, V = 6000, 9000
    print(f"pieces of {length} D={D} {gdt}", flush=True)
    base = np.repeat(np.arange((K + length - 1) // length) + 3, length)[:K].astype(np.int32)
    rng = np.random.Generator(np.random.PCG64(900 + length + D))
    ids = torch.from_numpy(rng.permutation(base)).to(DEV)
    grad = torch.from_numpy(rng.integers(-8, 9, (K, D))).to(DEV)
    want = torch.zeros((V, D), dtype=torch.int64, device=DEV).index_add_(0, ids.long(), grad).float()
    grad = grad.to(torch.bfloat16 if gdt == "bf16" else torch.float32)
    r = lz.unique(ids, V)
    seg = (grad, r.perm, r.inverse, r.offsets, r.num_unique)
    U = int(r.num_unique.item())
    ws = lz.Workspace(DEV)
    for _ in range(2):
        out = lz.segsum(*seg, dev_err=r.dev_err, ws=ws)
        assert torch.equal(out[:U], want[r.uniq[:U].long()])
    t = torch.zeros((V, D), device=DEV)
    lz.segsum_sgd(*seg, r.uniq, t, -1.0, dev_err=r.dev_err, ws=ws)
    assert torch.equal(t, want)
    p, m, v = (torch.zeros((V, D), device=DEV) for _ in range(3))
    lz.segsum_adam(*seg, r.uniq, p, m, v, lr=0.0, beta1=0.0, step=1, dev_err=r.dev_err, ws=ws)
    assert torch.equal(m, want)
    lz.check(r.dev_err)


@pytest.mark.parametrize("D,gdt", [(512, "f32"), (517, "f32"), (1100, "bf16")])
def test_words_that_the_call_before_left(lz, D, gdt):
    """Calls on one workspace, in turn over lists whose heads and cut segments of
    a few pieces end and start in the same chunks: every chunk's word holds a
    flag, a count or both from the call before. Rows of small whole numbers."""
    K, V = 6000, 500
    print(f"words of the call before D={D} {gdt}", flush=True)
    rng = np.random.Generator(np.random.PCG64(1000 + D))
    ws, calls = lz.Workspace(DEV), []
    for lengths in ((300, 40), (40, 300, 24), (24, 700)):
        n = np.resize(lengths, K)
        base = np.repeat(np.arange(K), n)[:K].astype(np.int32)
        ids = torch.from_numpy(rng.permutation(base)).to(DEV)
        grad = torch.from_numpy(rng.integers(-8, 9, (K, D))).to(DEV)
        want = torch.zeros((V, D), dtype=torch.int64, device=DEV).index_add_(0, ids.long(), grad)
        grad = grad.to(torch.bfloat16 if gdt == "bf16" else torch.float32)
        r = lz.unique(ids, V)
        calls.append((r, (grad, r.perm, r.inverse, r.offsets, r.num_unique), want.float()))
    outs = [(r, lz.segsum(*seg, dev_err=r.dev_err, ws=ws), want)
            for _ in range(4) for r, seg, want in calls]
    for r, out, want in outs:
        U = int(r.num_unique.item())
        assert torch.equal(out[:U], want[r.uniq[:U].long()])
        lz.check(r.dev_err)
