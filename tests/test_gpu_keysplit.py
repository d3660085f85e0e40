"""The key-split first pass (64 query rows a workgroup, a quarter of the keys a
wave), taken where a grid has at most 256 such units, or 512 over a long walk,
against whole 256-row tiles: the same slabs in a call just over the line.  The two sum the keys in
another order (and round each probability to fp16 alike), so bf16 outputs agree
to the rounding of the output, and nearly all are equal."""
import pytest
import torch

from paper_2609_35110_amd import sol

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    sol.lib()
    yield
    torch.cuda.synchronize()


def _slabs(rows):
    """The largest number of slabs of that many rows that splits, and one over."""
    n = 256 // -(-rows // 64)
    return n, n + 1


def _qkv(slabs, rows, keys, seed):
    gen = torch.Generator(DEV).manual_seed(seed)
    draw = lambda n: torch.randn((1, slabs, n, 128), generator=gen, device=DEV).bfloat16()
    return draw(rows), draw(keys), draw(keys)


def _check(split, whole, label):
    """The two start a tile's scores from -m or subtract m after, so a
    probability may round to the other fp16 neighbour, 2^-11 of itself: the
    outputs, means of v weighted by probabilities that sum to one, move by at
    most 2^-11 of a weighted mean of |v| (below 2 for these v); the row sums by
    2^-11 (fp16 word sums against fp32).  Then each is rounded to bf16: one
    step, at most 2^-7 of it."""
    a, b = split.float(), whole.float()
    bound = torch.maximum(a.abs(), b.abs()) * (2.0 ** -7 + 2.0 ** -11) + 2.0 ** -10
    assert bool(((a - b).abs() <= bound).all()), (label, float(((a - b).abs() - bound).max()))
    assert float((a == b).float().mean()) >= 0.9, label


# rows around a unit and a tile; keys around a tile, a block of four, and walks
# that leave waves without keys or with an odd number of tiles
SHAPES = [(64, 1), (1, 31), (63, 33), (65, 128), (64, 129), (257, 160), (300, 257), (100, 1000), (513, 700)]


@pytest.mark.parametrize("rows,keys", SHAPES)
def test_dense_equals_whole_tiles(rows, keys):
    n, over = _slabs(rows)
    q, k, v = _qkv(over, rows, keys, 100 * rows + keys)
    outs = []
    for s in (n, over):
        kp, vp = sol.prepared_kv_buffers(1, s, keys, DEV)
        sol.prepare_kv_ex(k[:, :s].contiguous(), v[:, :s].contiguous(), 0, 0, 0, None, kp, vp)
        outs.append(sol.attn_fwd_prepared_ex(q[:, :s].contiguous(), kp, vp, keys, 0, 0, 0))
    _check(outs[0], outs[1][:, :n], "%dx%d" % (rows, keys))


@pytest.mark.parametrize("fmt", ["fp8", "int8_records"])
def test_coded_outputs_equal_whole_tiles(fmt):
    """E4M3 codes and output records: codes differ only where a value lies
    within the two results' difference (~2e-4 of the RMS) of a midpoint; every
    byte of a record is written (the padding zero)."""
    rows, keys = 300, 700
    n, over = _slabs(rows)
    q, k, v = _qkv(over, rows, keys, 7)
    outs = []
    for s in (n, over):
        kp, vp = sol.prepared_kv_buffers(1, s, keys, DEV)
        sol.prepare_kv_ex(k[:, :s].contiguous(), v[:, :s].contiguous(), 0, 0, 0, None, kp, vp)
        shape = (1, s, rows, 128) if fmt == "fp8" else (1, rows, s, 144)
        out = torch.full(shape, 0x55, dtype=torch.uint8, device=DEV)
        outs.append(sol.attn_fwd_prepared_ex(q[:, :s].contiguous(), kp, vp, keys, 0, 0, 0, out=out, **{fmt: True}))
    a, b = outs[0], outs[1][:, :n] if fmt == "fp8" else outs[1][:, :, :n]
    if fmt == "int8_records":
        assert int(a[..., 132:].max()) == 0
        same = (a[..., 128:132] == b[..., 128:132]).all(-1)  # groups on the same scales
        assert float(same.float().mean()) >= 0.98
        a, b = a[..., :128].view(torch.int8).int(), b[..., :128].view(torch.int8).int()
        assert int((a - b).abs()[same].max()) <= 1
    assert float((a == b).float().mean()) >= 0.98


@pytest.mark.parametrize("tau", [-1e30, 0.5, 1e30])
def test_block_sparse_equals_whole_tiles(tau):
    """Lists of every length, a prefix across blocks, a ragged last block."""
    T, Hl, Wl, nt = 3, 11, 13, 300
    rows = nt + T * Hl * Wl
    n, over = _slabs(rows)
    q, k, v = _qkv(over, rows, rows, 11)
    tab = sol.rope3d_table(T, Hl, Wl, device=DEV)
    outs = []
    for s in (n, over):
        qs = q[:, :s].contiguous()
        kp, vp = sol.prepare_kv(k[:, :s].contiguous(), v[:, :s].contiguous(), T, Hl, Wl, tab)
        ws = sol.sparse_route(qs, kp, T, Hl, Wl, tab, tau)
        outs.append(sol.attn_fwd_sparse(qs, kp, vp, T, Hl, Wl, tab, ws))
    _check(outs[0], outs[1][:, :n], "sparse %g" % tau)


def test_overflowing_rows_go_to_the_second_pass():
    """Scores that peak 49 binades up in keys 200 to 400 -- neither the first
    tile nor the rows' diagonal one -- leave the fp16 range in one or two waves
    of a unit: its rows are recomputed, in every output format."""
    rows, keys = 130, 900
    n, over = _slabs(rows)
    q, k, v = _qkv(over, rows, keys, 13)
    q = torch.ones_like(q)
    at = torch.arange(keys, device=DEV)
    k = (k * 0.05 + 3 * torch.exp(-((at - 300) / 60.0) ** 2)[:, None]).bfloat16()
    for how in ({}, {"fp8": True}, {"int8_records": True}):
        outs = []
        for s in (n, over):
            kp, vp = sol.prepared_kv_buffers(1, s, keys, DEV)
            sol.prepare_kv_ex(k[:, :s].contiguous(), v[:, :s].contiguous(), 0, 0, 0, None, kp, vp)
            outs.append(sol.attn_fwd_prepared_ex(q[:, :s].contiguous(), kp, vp, keys, 0, 0, 0, **how))
        whole = outs[1][:, :, :n] if "int8_records" in how else outs[1][:, :n]
        assert torch.equal(outs[0], whole), how  # both are the second pass's


@pytest.mark.parametrize("keys", [1791, 1792, 2050])
def test_second_round_of_dense_units(keys):
    """257 to 512 units split from 1,792 keys on, 256 always, 513 never: a call of
    whole tiles has the bits of any other, one of split units others."""
    rows = 513  # 9 units a slab
    q, k, v = _qkv(57, rows, keys, keys)
    outs = {}
    for s in (28, 29, 56, 57):
        kp, vp = sol.prepared_kv_buffers(1, s, keys, DEV)
        sol.prepare_kv_ex(k[:, :s].contiguous(), v[:, :s].contiguous(), 0, 0, 0, None, kp, vp)
        outs[s] = sol.attn_fwd_prepared_ex(q[:, :s].contiguous(), kp, vp, keys, 0, 0, 0)
    for s in (28, 29, 56):
        whole = outs[57][:, :s]
        assert torch.equal(outs[s], whole) == (s != 28 and keys < 1792), s
        _check(outs[s], whole, "%d slabs, %d keys" % (s, keys))


@pytest.mark.parametrize("tokens,split,whole", [(300, 51, 52), (1800, 17, 18)])
def test_records_equal_whole_tiles(tokens, split, whole):
    """Queries, keys and values from records: one round of split units (255 of
    them) and two (493), against whole tiles (260, 522)."""
    q, k, v = _qkv(whole, tokens, tokens, tokens)
    outs = []
    for s in (split, whole):
        rec = sol.qkv_encode(*(x[:, :s].contiguous() for x in (q, k, v)))
        kp, vp = sol.prepared_kv_buffers(1, s, tokens, DEV)
        sol.prepare_kv_records(rec, kp, vp)
        outs.append(sol.attn_fwd_records(rec, kp, vp))
    assert not torch.equal(outs[0], outs[1][:, :split])
    _check(outs[0], outs[1][:, :split], "records, %d tokens" % tokens)


def _sparse(slabs, grid, text, tau, seed):
    rows = text + grid[0] * grid[1] * grid[2]
    q, k, v = _qkv(max(slabs), rows, rows, seed)
    tab = sol.rope3d_table(*grid, device=DEV)
    outs = []
    for s in slabs:
        qs = q[:, :s].contiguous()
        kp, vp = sol.prepare_kv(k[:, :s].contiguous(), v[:, :s].contiguous(), *grid, tab)
        ws = sol.sparse_route(qs, kp, *grid, tab, tau)
        outs.append(sol.attn_fwd_sparse(qs, kp, vp, *grid, tab, ws))
    return outs


# (slabs in two rounds, slabs over them, grid, prefix rows, split)
LISTED = [(12, 16, (3, 21, 33), 0, False),   # 2,079 tokens, 33 units a slab
          (12, 16, (3, 21, 32), 63, True),   # as many, a prefix: its query block walks every key
          (2, 3, (11, 1, 1117), 0, False),   # 12,287 tokens, 192 units a slab
          (2, 3, (12, 32, 32), 0, True)]     # 12,288


@pytest.mark.parametrize("two,over,grid,text,split", LISTED, ids=[str(c) for c in LISTED])
def test_second_round_of_block_sparse_units(two, over, grid, text, split):
    """257 to 512 units of a block-sparse call split only where some query block
    walks every key or the lists are long: elsewhere whole tiles are faster,
    and the call gives the bits of one past 512 units."""
    a, b = _sparse((two, over), grid, text, 1.0, 17)
    b = b[:, :two]
    assert torch.equal(a, b) != split
    _check(a, b, "%s + %d" % (grid, text))


def test_a_slab_on_either_side_of_the_line():
    """A slab's result is a function of its own data and of the form the call's
    sizes choose: bit for bit the same in every call of one form, whatever its
    neighbours, and across the line within the rounding of the output."""
    grid, text = (3, 11, 13), 37  # 466 tokens, 8 units a slab
    n, over = _slabs(text + grid[0] * grid[1] * grid[2])
    q, k, v = _qkv(over + 9, text + grid[0] * grid[1] * grid[2], text + grid[0] * grid[1] * grid[2], 23)
    tab = sol.rope3d_table(*grid, device=DEV)

    def run(at):
        return sol.attn_fwd_ws(*(x[:, at].contiguous() for x in (q, k, v)), *grid, tab)

    split = {(a, b): run(slice(a, b)) for a, b in ((0, n), (5, 6), (4, 9))}
    whole = {(a, b): run(slice(a, b)) for a, b in ((0, over), (3, over + 9))}
    for form, size in ((split, n), (whole, over)):
        for (first, end), out in form.items():
            end = min(end, size)
            assert torch.equal(out[:, :end - first], form[0, size][:, first:end]), (first, end)
    a, b = split[0, n], whole[0, over][:, :n]
    assert not torch.equal(a, b)
    _check(a, b, "across the line")
