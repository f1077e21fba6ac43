"""The toy "clean views" stage of the library (fbx_clean_*) against its oracle, byte for byte, and
cleaned text handed on to fbx_extract without leaving the device."""
import random

import numpy as np
import pytest

from oracle import fbx_clean_oracle as C
from oracle import fbx_oracle as O
from paper_2210_07768_amd import binding as B
from gpu_harness import assert_same, expand, to_device
from test_clean_oracle_pins import SPEC

pytestmark = pytest.mark.gpu


def _cat(records):
    return np.frombuffer(b"".join(records), np.uint8), np.cumsum([0] + [len(r) for r in records]).astype(np.uint64)


def _gpu_clean(spec, raw, off, out_cap=None, misalign=0, scratch_bytes=None):
    import torch
    n = len(off) - 1
    clean = B.Clean(spec)
    d_raw, d_off = to_device(raw, off, misalign)
    scratch = torch.empty(scratch_bytes or clean.scratch_hint(n), dtype=torch.uint8, device="cuda").fill_(0x6B)
    d_out = torch.empty(raw.size + 64 * n + 64 if out_cap is None else out_cap, dtype=torch.uint8, device="cuda").fill_(0x21)
    d_out_off = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
    res = clean.run(d_raw, d_off, d_out, d_out_off, scratch)
    clean.close()
    return res, d_out, d_out_off


def _random_case(rng, n):
    F = rng.randint(1, 6)
    lines = ["fbxclean 1", f"fields {F}"]
    for _ in range(rng.randint(0, 7)):
        kind = rng.choice(["fill", "key", "keep"])
        arg = "".join(rng.choice("abck") for _ in range(rng.randint(0 if kind != "fill" else 1, 2))).encode().hex()
        lines.append(f"{kind} field={rng.randrange(F)} {dict(fill='value', key='name', keep='prefix')[kind]}={arg}")
    field = lambda: "".join(rng.choice("abc:;k") for _ in range(rng.randint(0, 12)))
    recs = [("\t".join(field() for _ in range(rng.randint(0, F + 1))) + ("\n" if rng.random() < 0.7 else "")).encode()
            for _ in range(n)]
    return "\n".join(lines) + "\n", recs


@pytest.mark.parametrize("seed", range(8))
def test_clean_matches_the_oracle(seed):
    rng = random.Random(100 + seed)
    spec, recs = _random_case(rng, rng.choice([1, 255, 256, 257, 5000]))
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(spec, raw, off)
    res, d_out, d_out_off = _gpu_clean(spec, raw, off, misalign=seed % 3)
    assert res.n_kept == len(want_off) - 1 and res.out_len == want_raw.size
    assert np.array_equal(d_out_off[:res.n_kept + 1].cpu().numpy().view(np.uint64), want_off)
    assert np.array_equal(d_out[:res.out_len].cpu().numpy(), want_raw)
    assert bool((d_out[res.out_len:] == 0x21).all()), "written beyond the cleaned text"


def _wide_case(rng, F, n, long_every=0, n_ops=12, width=10, keep_all=False):
    """n records of about F fields (some fewer, some more) of 0..width bytes, operators on random fields;
    every long_every-th record holds one field of 30 to 70 KB."""
    lines = ["fbxclean 1", f"fields {F}"]
    for o in range(n_ops):
        kind = "keep" if o == n_ops // 2 else rng.choice(["fill", "fill", "key"])  # (one filter: more would drop nearly every record)
        arg = "".join(rng.choice("abk") for _ in range(rng.randint(0 if kind != "fill" else 1, {"fill": 9, "key": 2, "keep": 0 if keep_all else 1}[kind]))).encode().hex()
        lines.append(f"{kind} field={rng.randrange(F)} {dict(fill='value', key='name', keep='prefix')[kind]}={arg}")
    field = lambda: "".join(rng.choice("abc:;k") for _ in range(rng.randint(0, width)))
    recs = []
    for i in range(n):
        fields = [field() for _ in range(F + rng.choice([0, 0, 0, 0, -1, 1, -F // 2]))]
        if long_every and i % long_every == long_every - 1 and fields:
            fields[rng.randrange(len(fields))] = "".join(rng.choice("ab;:k") for _ in range(64)) * rng.randint(470, 1100)
        recs.append(("\t".join(fields) + ("\n" if rng.random() < 0.8 else "")).encode())
    return "\n".join(lines) + "\n", recs


@pytest.mark.parametrize("F,n,long_every,n_ops,width", [
    (130, 3000, 0, 40, 10),      # tiles of 16 records, two turns of a wavefront per record
    (130, 3001, 0, 40, 10),      # the same with a filter that keeps every record
    (100, 2500, 97, 30, 8),      # now and then a tile whose text does not fit the section: read in place
    (1, 9000, 0, 2, 6),          # tiles of 64 short records
    (7, 700, 5, 6, 300),         # long fields: few records per tile, many tiles read in place
    (5000, 24, 0, 50, 3),        # more fields than the tables of the kernel without segments hold: a record per thread
    (20000, 5, 0, 50, 3),        # more than any table in LDS holds
    (100, 900, 50, 2500, 6),     # more operators than LDS holds beside the text: no segments are kept
])
@pytest.mark.parametrize("keep", [True, False])
def test_clean_tiles_of_every_shape(F, n, long_every, n_ops, width, keep):
    """keep: with room for segments in the scratch buffer (where the specification allows it), or with 24 bytes a record."""
    rng = random.Random(F * 1000 + n)
    spec, recs = _wide_case(rng, F, n, long_every, n_ops, width, keep_all=n % 2 == 1)
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(spec, raw, off)
    assert 0 < len(want_off) - 1, "the case keeps no record"
    little = 24 * n + 16 * n_ops + 4 * F + 9 * n_ops + 3 * 4096  # (records; operators, fields and arguments; alignment)
    res, d_out, d_out_off = _gpu_clean(spec, raw, off, out_cap=want_raw.size + 1000, misalign=n % 5, scratch_bytes=None if keep else little)
    assert res.n_kept == len(want_off) - 1 and res.out_len == want_raw.size
    assert np.array_equal(d_out_off[:res.n_kept + 1].cpu().numpy().view(np.uint64), want_off)
    assert np.array_equal(d_out[:res.out_len].cpu().numpy(), want_raw)
    assert bool((d_out[res.out_len:] == 0x21).all()), "written beyond the cleaned text"


@pytest.mark.parametrize("n", [1, 3, 64, 65, 127, 500])
@pytest.mark.parametrize("kept", ["none", "first", "last", "every_fourth", "runs", "all"])
def test_clean_keeps_few_many_or_all_records_of_a_tile(n, kept):
    """Which records of a tile of 64 stay, with records of no bytes, of less than a chunk, and of more than 64 chunks."""
    rng = random.Random(n)
    stays = {"none": lambda i: False, "first": lambda i: i % 64 == 0, "last": lambda i: i % 64 == 63 or i == n - 1, "every_fourth": lambda i: i % 4 == 2,
             "runs": lambda i: i // 5 % 3 == 0, "all": lambda i: True}[kept]
    recs = [b"" if kept == "all" and i % 7 == 3 else
            (("k" if stays(i) else "d") + "x" * (rng.randint(1000, 1400) if i % 40 == 9 else rng.randint(0, 20)) + "\t" + "y" * rng.randint(0, 3) + "\n").encode()
            for i in range(n)]
    spec = "fbxclean 1\nfields 2\nfill field=1 value=6e6f6e65\n" + ("" if kept == "all" else "keep field=0 prefix=6b\n")
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(spec, raw, off)
    for misalign in (0, 7):
        res, d_out, d_out_off = _gpu_clean(spec, raw, off, out_cap=want_raw.size + 64, misalign=misalign)
        assert res.n_kept == len(want_off) - 1 and res.out_len == want_raw.size
        assert np.array_equal(d_out_off[:res.n_kept + 1].cpu().numpy().view(np.uint64), want_off)
        assert np.array_equal(d_out[:res.out_len].cpu().numpy(), want_raw)
        assert bool((d_out[res.out_len:] == 0x21).all()), "written beyond the cleaned text"


def test_a_scratch_buffer_without_room_for_segments_still_does():
    """24 bytes a record and the tables: too little to keep segments, enough for the kernel that keeps none."""
    import torch
    n = 1000
    spec = ("fbxclean 1\nfields 100\n" + "".join(f"fill field={k} value=30\n" for k in range(30))
            + "key field=40 name=6b31\nkeep field=5 prefix=61\n")
    rng = random.Random(5)
    recs = [("\t".join("" if rng.random() < 0.3 else rng.choice(["a1", "b", "k1:x;k2:y"]) for _ in range(100)) + "\n").encode() for _ in range(n)]
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(spec, raw, off)
    clean = B.Clean(spec)
    d_raw, d_off = to_device(raw, off, 3)
    hint = clean.scratch_hint(n)
    tables = 512 + 512 + 256  # 32 operators of 16 bytes, 101 words, the arguments: each in whole 256 bytes
    little = 2 * 256 + tables + 8192 + 16128 + 256
    assert little < hint
    for size in (little, hint - 256, hint):
        d_out = torch.empty(want_raw.size + 64, dtype=torch.uint8, device="cuda").fill_(0x21)
        d_out_off = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
        buf = torch.empty(size + 256, dtype=torch.uint8, device="cuda").fill_(0x6B)
        res = clean.run(d_raw, d_off, d_out, d_out_off, buf[:size])
        assert res.n_kept == len(want_off) - 1 and res.out_len == want_raw.size
        assert np.array_equal(d_out_off[:res.n_kept + 1].cpu().numpy().view(np.uint64), want_off)
        assert np.array_equal(d_out[:res.out_len].cpu().numpy(), want_raw)
        assert bool((buf[size:] == 0x6B).all()), "written beyond the scratch buffer"
        note = B.lib().fbx_clean_last_error(clean._h).decode()
        assert str(hint) in note if size < hint else note == ""
    with pytest.raises(B.FbxError) as e:
        clean.run(d_raw, d_off, d_out, d_out_off, buf[:little // 2])
    assert e.value.status == B.E_NOMEM
    clean.close()


def test_clean_edge_cases_and_errors():
    import torch
    recs = [b"ann\tage:3;city:rome;x:1\tok1\t5\n", b"\tcity:;age:4\tokay\t\n", b"bob\tage:3\tok\t1", b"cy\tcity:oslo\tnot ok\t2\n",
            b"", b"\t\tok\t\n"] * 100
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(SPEC, raw, off)
    # an empty batch
    res, d_out, d_out_off = _gpu_clean(SPEC, raw[:0], off[:1])
    assert res.n_kept == 0 and res.out_len == 0 and int(d_out_off[0]) == 0
    # an output buffer that is too small: nothing written, the need reported, and that much suffices
    with pytest.raises(B.FbxError) as e:
        _gpu_clean(SPEC, raw, off, out_cap=want_raw.size - 1)
    assert e.value.status == B.E_NOMEM and e.value.required_bytes == want_raw.size
    res, d_out, d_out_off = _gpu_clean(SPEC, raw, off, out_cap=want_raw.size)
    assert np.array_equal(d_out.cpu().numpy(), want_raw)
    # scratch too small, bad offsets, bad spec
    clean = B.Clean(SPEC)
    d_raw, d_off = to_device(raw, off)
    d_out = torch.empty(raw.size * 2, dtype=torch.uint8, device="cuda")
    d_out_off = torch.empty(len(recs) + 1, dtype=torch.int64, device="cuda")
    with pytest.raises(B.FbxError) as e:
        clean.run(d_raw, d_off, d_out, d_out_off, torch.empty(1024, dtype=torch.uint8, device="cuda"))
    assert e.value.status == B.E_NOMEM
    bad = off.copy(); bad[7] = bad[9]
    d_raw2, d_off2 = to_device(raw, bad)
    with pytest.raises(B.FbxError) as e:
        clean.run(d_raw2, d_off2, d_out, d_out_off, torch.empty(clean.scratch_hint(len(recs)), dtype=torch.uint8, device="cuda"))
    assert e.value.status == B.E_INPUT
    clean.close()
    for spec in ("fields 2\n", "fbxclean 1\nfields 2\nfill field=2 value=61\n", "fbxclean 1\nfields 2\nfill field=0 value=09\n",
                 "fbxclean 1\nfields 2\nkeep field=0\n", "fbxclean 1\nfields 2\nfrob field=0 value=61\n"):
        with pytest.raises(B.FbxError) as e:
            B.Clean(spec)
        assert e.value.status == B.E_SPEC


def test_cleaned_text_feeds_extraction_on_the_device():
    """Clean, then extract, both on the device, against the two oracles chained on the host."""
    import torch
    rng = random.Random(77)
    word = lambda: "".join(rng.choice("abcdxyz") for _ in range(rng.randint(1, 8)))
    recs = []
    for i in range(4000):
        attrs = ";".join(f"{k}:{word()}" for k in rng.sample(["city", "age", "tag", "os"], rng.randint(0, 4)))
        terms = ",".join(word() for _ in range(rng.randint(1, 5))) if i % 9 else ""
        price = f"{rng.randint(0, 300)}.{rng.randint(0, 99)}" if i % 7 else ""
        recs.append(f"{word() if i % 5 else ''}\t{attrs}\t{terms}\t{price}\t{rng.choice(['click', 'view', 'skip'])}\n".encode())
    clean_spec = ("fbxclean 1\nfields 5\n"
                  f"fill field=0 value={b'anon'.hex()}\n"
                  f"key field=1 name={b'city'.hex()}\n"
                  f"fill field=1 value={b'nowhere'.hex()}\n"
                  f"fill field=2 value={b'none'.hex()}\n"
                  f"fill field=3 value={b'0'.hex()}\n"
                  f"keep field=4 prefix={b'cli'.hex()}\n")
    extract_spec = ("fbx 1\nfields 5\n"
                    "op u hash slot=0 seed=1 emit=1 field=0 multi=0\n"
                    "op c hash slot=1 seed=2 emit=1 field=1 multi=0\n"
                    "op t hash slot=2 seed=3 emit=1 field=2 multi=1\n"
                    "op p bucket slot=3 seed=4 emit=1 field=3 multi=0 bounds=1000000,10000000,100000000\n"
                    "op uc cross slot=4 seed=5 emit=1 a=u b=c\n"
                    "op ct cross slot=5 seed=6 emit=1 a=c b=t\n")
    raw, off = _cat(recs)
    want_raw, want_off = C.clean(clean_spec, raw, off)
    want = O.extract(extract_spec, want_raw, want_off)
    assert 0 < len(want_off) - 1 < len(recs) and want.n_malformed_numeric == 0
    res, d_out, d_out_off = _gpu_clean(clean_spec, raw, off)
    plan = B.Plan(extract_spec)
    got, ws = B.extract_with_retry(plan, d_out[:res.out_len], d_out_off[:res.n_kept + 1])
    assert_same({s: expand(got.slots[s], res.n_kept) for s in got.slot_ids}, got, want, "clean then extract")
    plan.close()


def test_threads_share_a_specification():
    """Calls that run at the same time on one specification, with buffers of their own, get their own sizes back."""
    import threading

    import torch
    spec = "fbxclean 1\nfields 3\nfill field=1 value=30\nkeep field=0 prefix=61\n"
    clean = B.Clean(spec)
    rng = random.Random(8)
    cases = []
    for n in (40, 700, 3, 1500):  # (from one tile to many: calls of different lengths)
        raw, off = _cat([(rng.choice("ab") + "\t" + rng.choice(["", "x"]) + "\tend\n").encode() for _ in range(n)])
        want_raw, want_off = C.clean(spec, raw, off)
        d_raw, d_off = to_device(raw, off)
        cases.append((d_raw, d_off, len(want_off) - 1, want_raw, torch.empty(want_raw.size + 64, dtype=torch.uint8, device="cuda"),
                      torch.empty(n + 1, dtype=torch.int64, device="cuda"),
                      torch.empty(clean.scratch_hint(n), dtype=torch.uint8, device="cuda"), torch.cuda.Stream()))
    torch.cuda.synchronize()
    wrong = []

    def calls(d_raw, d_off, n_kept, want, d_out, d_out_off, scratch, stream):
        for i in range(300):
            res = clean.run(d_raw, d_off, d_out, d_out_off, scratch, stream=stream.cuda_stream)
            if (res.n_kept, res.out_len) != (n_kept, want.size):
                wrong.append((i, res.n_kept, n_kept, res.out_len, want.size))
                return

    threads = [threading.Thread(target=calls, args=c) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
    for d_raw, d_off, n_kept, want, d_out, *_ in cases:
        assert np.array_equal(d_out[:want.size].cpu().numpy(), want)
    clean.close()
