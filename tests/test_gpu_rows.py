"""GPU parity of the masking of logits rows at every alignment: a row is cut
at 128-byte lines of memory into 4 KiB tiles, so its first and last tile, the
lines at their ends, lines masked whole and lines left alone are the cases;
large batches read, select and write densely mixed tiles instead; short rows,
small batches and logits off their own alignment are masked an element per
thread.  Compared bit for bit with the closed form on the same bits (the apply only copies or
writes -inf)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2608_03065_amd import psc  # noqa: E402
from paper_2608_03065_amd.psc import Classifier, DecodeStates, apply_mask, pack_states  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _mixed_bits(B, W, seed):
    """Runs of words all masked, all allowed, sparsely masked and dense."""
    g = torch.Generator(DEV).manual_seed(seed)
    word = lambda: torch.randint(-2**31, 2**31, (B, W), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
    kind = torch.randint(0, 4, (B, (W + 6) // 7), generator=g, device=DEV).repeat_interleave(7, 1)[:, :W]
    sparse = ~(word() & word() & word() & word())
    return torch.where(kind == 0, 0, torch.where(kind == 1, -1, torch.where(kind == 2, sparse, word()))).int()


def _check(B, V, dtype, offset, bits):
    ints = torch.int16 if dtype == torch.bfloat16 else torch.int32
    buf = torch.randint(-2**15, 2**15, (offset + B * V + 80,), device=DEV, dtype=torch.int32).to(ints)
    want = buf.clone()
    rows = want[offset:offset + B * V].view(B, V)
    inf = torch.tensor(float("-inf"), dtype=dtype).view(ints).item()
    shift = torch.arange(32, device=DEV, dtype=torch.int32)
    part = max(8, 2**24 // V)
    for b0 in range(0, B, part):       # in parts: the expanded bits are 4 bytes each
        allowed = ((bits[b0:b0 + part, :, None] >> shift) & 1).bool().flatten(1)[:, :V]
        rows[b0:b0 + part].masked_fill_(~allowed, inf)
    apply_mask(buf.view(dtype)[offset:offset + B * V].view(B, V), bits)
    torch.cuda.synchronize()
    assert torch.equal(buf, want), (B, V, dtype, offset)   # also what lies before and after the rows


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [31, 511, 512, 513, 1023, 1025, 2047, 2048, 2049, 2111, 4096, 4160, 6145])
def test_rows_at_every_alignment(V, dtype):
    line, item = (64, 2) if dtype == torch.bfloat16 else (32, 4)
    many = (3 << 19) // (V * item) + line     # rows past the size below which elements are masked one by one
    for offset in (0, 1, 7, line // 2, line - 1):
        for B in (line + 3, many):
            _check(B, V, dtype, offset, _mixed_bits(B, (V + 31) // 32, V + offset))


@pytest.mark.parametrize("dtype,B,V", [(torch.bfloat16, 3, 262143), (torch.bfloat16, 3, 262145),
                                       (torch.bfloat16, 768, 1024), (torch.bfloat16, 767, 1024),
                                       (torch.float32, 3, 131071), (torch.float32, 3, 131073),
                                       (torch.float32, 1, 393216), (torch.float32, 1, 393184)])
def test_apply_around_the_small_batch_limit(dtype, B, V):
    """Batches below 1.5 MiB are masked an element per thread, larger ones by
    tiles."""
    for offset in (0, 1):
        _check(B, V, dtype, offset, _mixed_bits(B, (V + 31) // 32, V))


@pytest.mark.parametrize("dtype,B,V,offset", [(torch.bfloat16, 28, 2000001, 5), (torch.bfloat16, 27, 2097152, 0),
                                              (torch.float32, 27, 1050001, 3), (torch.bfloat16, 22, 2097152, 0),
                                              (torch.bfloat16, 23, 2097152, 64), (torch.bfloat16, 24, 2000003, 1),
                                              (torch.float32, 25, 1048576, 0), (torch.float32, 26, 1048577, 1)])
def test_large_batch_dense_and_sparse(dtype, B, V, offset):
    """Above 88 (bf16) and 100 (fp32) MiB of logits dense rows are read,
    selected and written, sparse ones and the first and last tiles of a row are
    stored; batches of those sizes and just past them."""
    W = (V + 31) // 32
    bits = _mixed_bits(B, W, 3)
    dense = torch.randint(-2**31, 2**31, (B // 2, W), device=DEV, dtype=torch.int64).to(torch.int32)
    bits[:B // 2] = dense
    _check(B, V, dtype, offset, bits)


@pytest.mark.parametrize("V,B", [(513, 2**26 + 4101), (544, 2**22 + 5), (480, 2**23 + 3), (33, 2**26 + 77)])
def test_apply_past_one_launch(V, B):
    """More wavefronts than one launch can hold (rows of 513: 69 GB), and more
    elements than 31 bits count, of rows of whole mask words and of short ones.
    The masks have a period of 64 rows, so every 2^20 rows end the same."""
    torch.cuda.empty_cache()
    W, dtype, part = (V + 31) // 32, torch.bfloat16, 2**20
    period = _mixed_bits(64, W, V)
    bits = period.repeat((B + 63) // 64, 1)[:B]
    logits = torch.zeros(B, V, dtype=torch.int16, device=DEV)
    apply_mask(logits.view(dtype), bits)
    shift = torch.arange(32, device=DEV, dtype=torch.int32)
    allowed = ((period[:, :, None] >> shift) & 1).bool().flatten(1)[:, :V]
    inf = torch.tensor(float("-inf"), dtype=dtype).view(torch.int16).item()
    want = torch.zeros(64, V, dtype=torch.int16, device=DEV).masked_fill_(~allowed, inf).repeat(part // 64, 1)
    for b in range(0, B, part):
        assert torch.equal(logits[b:b + part], want[:min(part, B - b)]), (V, b)
    del logits, bits, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 33), (torch.bfloat16, 513), (torch.bfloat16, 3071),
                                     (torch.bfloat16, 3072), (torch.bfloat16, 3073), (torch.float32, 513),
                                     (torch.float32, 1535), (torch.float32, 1536), (torch.float32, 1537)])
@pytest.mark.parametrize("layout", ["flat", "sliced"])
def test_step_rows_around_the_element_limit(dtype, V, layout):
    """Rows below 6 KiB are masked an element per thread, longer ones by tiles:
    the same logits and bitmask as the host walk's masks, at odd offsets."""
    class Vocab:
        tokens = [b"%d" % (10 + i) if i % 3 else b"x%d" % i for i in range(V - 1)] + [b""]
        eos_id = V - 1
    clf = Classifier.from_text('%start v\nN: /[0-9]+/\nS: /"[a-z0-9]*"/\nv: N | S\n', Vocab).bind(DEV, layout=layout)
    states = [clf.host_state(t) for t in (b"", b'"', b"12", b'"a"')] * 17
    bits = torch.from_numpy(clf.masks_host(states).view("int32")).to(DEV)
    ints = torch.int16 if dtype == torch.bfloat16 else torch.int32
    shift = torch.arange(32, device=DEV, dtype=torch.int32)
    allowed = ((bits[:, :, None] >> shift) & 1).bool().flatten(1)[:, :V]
    inf = torch.tensor(float("-inf"), dtype=dtype).view(ints).item()
    for offset in (0, 1, 16):
        n = len(states) * V
        buf = torch.randint(-2**15, 2**15, (offset + n + 80,), device=DEV, dtype=torch.int32).to(ints)
        want = buf.clone()
        want[offset:offset + n].view(-1, V).masked_fill_(~allowed, inf)
        out = torch.empty_like(bits)
        clf.compute_and_apply(*pack_states(states, DEV), buf.view(dtype)[offset:offset + n].view(-1, V), out=out)
        assert torch.equal(buf, want) and torch.equal(out, bits), offset


@pytest.mark.parametrize("dtype,B", [(torch.bfloat16, 219), (torch.bfloat16, 220), (torch.float32, 124),
                                     (torch.float32, 125)])
def test_step_of_large_batches(dtype, B):
    """The step and the decoding step (two launches) on either side of the size
    from which dense tiles are read, selected and written, rows of 210,001 at
    an odd offset, masks dense (every token or two of three) and sparse."""
    V = 210001

    class Vocab:
        tokens = [b"%d" % (10 + i) if i % 3 else b"x%d" % i for i in range(V - 1)] + [b""]
        eos_id = V - 1
    clf = Classifier.from_text('%start v\nN: /[0-9]+/\nS: /"[a-z0-9]*"/\nv: N | S\n', Vocab).bind(DEV)
    kinds = [clf.host_state(t) for t in (b"", b'"', b"12", b'"a"')]
    states = [kinds[b % 4] for b in range(B)]
    bits = torch.from_numpy(clf.masks_host(kinds).view("int32")).to(DEV)
    shift = torch.arange(32, device=DEV, dtype=torch.int32)
    masked = ~((bits[:, :, None] >> shift) & 1).bool().flatten(1)[:, :V]
    bits, masked = bits[torch.arange(B) % 4], masked[torch.arange(B) % 4]
    ints = torch.int16 if dtype == torch.bfloat16 else torch.int32
    inf = torch.tensor(float("-inf"), dtype=dtype).view(ints).item()
    old = torch.randint(-2**15, 2**15, (B * V + 81,), device=DEV, dtype=torch.int32).to(ints)
    want = old.clone()
    want[1:1 + B * V].view(B, V).masked_fill_(masked, inf)
    ds = DecodeStates(clf, B, 16, DEV).load(states)
    skip = torch.full((B,), -1, dtype=torch.int32, device=DEV)
    for call in (lambda lg, out: clf.compute_and_apply(*pack_states(states, DEV), lg, out=out),
                 lambda lg, out: ds.decode_step(skip, lg, out=out)):
        buf, out = old.clone(), torch.empty_like(bits)
        call(buf.view(dtype)[1:1 + B * V].view(B, V), out)
        assert torch.equal(buf, want) and torch.equal(out, bits)


@pytest.mark.parametrize("dtype,skew", [(torch.bfloat16, 1), (torch.float32, 1), (torch.float32, 2)])
@pytest.mark.parametrize("V,B", [(33, 70), (513, 2500), (5001, 40), (5001, 1100), (40001, 9)])
def test_logits_off_their_own_alignment(V, B, dtype, skew):
    """Logits at a byte address that is no multiple of their element's size, as
    only a C caller can hand over: the apply, the step, both forms of the
    decoding step (batches of at most 2,048 workgroups and larger ones) and the
    argmax, an element per thread at every size."""
    class Vocab:
        tokens = [b"%d" % (10 + i) if i % 3 else b"x%d" % i for i in range(V - 1)] + [b""]
        eos_id = V - 1
    clf = Classifier.from_text('%start v\nN: /[0-9]+/\nS: /"[a-z0-9]*"/\nv: N | S\n', Vocab).bind(DEV)
    kinds = [clf.host_state(t) for t in (b"", b'"', b"12", b'"a"')]
    states = [kinds[b % 4] for b in range(B)]
    bits = torch.from_numpy(clf.masks_host(kinds).view("int32")).to(DEV)[torch.arange(B) % 4]
    item, code = (2, psc.PSC_BF16) if dtype == torch.bfloat16 else (4, psc.PSC_F32)
    ints = torch.int16 if dtype == torch.bfloat16 else torch.int32
    shift = torch.arange(32, device=DEV, dtype=torch.int32)
    allowed = ((bits[:, :, None] >> shift) & 1).bool().flatten(1)[:, :V]
    x = torch.randn(B, V, device=DEV).to(dtype)
    want = x.masked_fill(~allowed, float("-inf"))
    packed = pack_states(states, DEV)
    ds, spare = DecodeStates(clf, B, 16, DEV).load(states), DecodeStates(clf, B, 16, DEV)
    skip = torch.full((B,), -1, dtype=torch.int32, device=DEV)
    out, toks = torch.empty_like(bits), torch.empty(B, dtype=torch.int32, device=DEV)
    ptr = lambda *ts: [t.data_ptr() for t in ts]
    st, n = ptr(*packed), B * V * item
    calls = {
        "apply": lambda p: psc.lib().psc_apply_mask(p, code, bits.data_ptr(), B, V, None),
        "step": lambda p: psc.lib().psc_compute_and_apply(clf._h, *st, B, out.data_ptr(), p, code, V, None),
        "decode": lambda p: psc.lib().psc_decode_step(
            clf._h, *ptr(ds.stacks, ds.lens, ds.qs, spare.stacks, spare.lens, spare.qs), 16, B,
            *ptr(skip, ds.status, out), p, code, V, None),
        "argmax": lambda p: psc.lib().psc_compute_and_argmax(clf._h, *st, B, p, code, V, toks.data_ptr(), None)}
    for name, call in calls.items():
        buf = torch.full((skew + n + 64,), 0x5A, dtype=torch.uint8, device=DEV)
        buf[skew:skew + n] = x.view(torch.uint8).flatten()
        out.zero_()
        torch.cuda.synchronize()
        psc._check(call(buf.data_ptr() + skew))
        torch.cuda.synchronize()
        got = buf[skew:skew + n].clone().view(ints).view(B, V)
        assert torch.equal(got, (x if name == "argmax" else want).view(ints)), name
        assert (buf[:skew] == 0x5A).all() and (buf[skew + n:] == 0x5A).all(), name
        if name in ("step", "decode"):
            assert torch.equal(out, bits), name
    f = want.float()
    best = f.max(1, keepdim=True).values
    first = torch.where((f == best) & allowed, torch.arange(V, device=DEV), V).amin(1)
    assert torch.equal(toks.long(), torch.where(allowed.any(1), first, -1))
