"""GPU parity: libfbx (through the C ABI) against the CPU oracle, bit-exact.
All arithmetic on the path is integer, so the tolerance is zero."""
import random

import numpy as np
import pytest

from oracle import fbx_oracle as O
from paper_2210_07768_amd import binding as B
from paper_2210_07768_amd import workloads as W
from helpers import FOLLOW_SPEC, FRAMING_RECORDS, FRAMING_SPEC, random_dag
from gpu_harness import assert_same, check, check_window, device_workload, expand, run_gpu, to_device
from oracle_ranges import check_every_sign, extract_parallel

pytestmark = pytest.mark.gpu

MODES = [{"fused": 0}, {"fused": 1}]
# the tile kernel at forced tile sizes and with a small staging section, so that tiles take
# several passes and some records are read in place
TILE_MODES = [{"tile_log2": 6}, {"tile_log2": 4}, {"tile_log2": 2, "raw_cap": 2048}, {"tile_log2": 0},
              {"tile_log2": 5, "raw_cap": 512}, {"tile_log2": 3, "raw_cap": 64}]
TILE_IDS = ["T64", "T16", "T4_cap2048", "T1", "T32_cap512", "T8_cap64"]


def _cat(records):
    raw = b"".join(records)
    off = np.cumsum([0] + [len(r) for r in records]).astype(np.uint64)
    return raw, off


@pytest.mark.parametrize("mode", MODES, ids=["per_layer", "fused"])
@pytest.mark.parametrize("copies", [1, 7, 29])
def test_hand_built_records(mode, copies):
    # 9, 63 and 261 records: less than a tile, one short of a tile, several tiles and a ragged tail
    raw, off = _cat(FRAMING_RECORDS * copies)
    check(FRAMING_SPEC, raw, off, mode)


@pytest.mark.parametrize("mode", MODES, ids=["per_layer", "fused"])
@pytest.mark.parametrize("cfg,n", [(1, 4096), (2, 700), (3, 3001), (4, 1500), (5, 2050)])
def test_configs_small(cfg, n, mode):
    w = W.get(cfg, n)
    raw, off = w.generate()
    res, want = check(w.spec, raw, off, mode, label=w.name)
    assert res.n_layers == w.n_layers


@pytest.mark.parametrize("mode", TILE_MODES, ids=TILE_IDS)
def test_tile_sizes_passes_and_in_place_records(mode):
    raw, off = _cat(FRAMING_RECORDS * 29)
    check(FRAMING_SPEC, raw, off, mode, label="framing")
    for cfg, n in ((5, 300), (2, 90), (3, 500), (4, 260)):
        w = W.get(cfg, n)
        raw, off = w.generate()
        check(w.spec, raw, off, mode, label=f"{w.name} {mode}")


# crosses of a multi-valued hash with a single sign, which the tile kernel computes along with
# the hash's items: the hash on either side, emitted or not, the single sign from layer 1 or from
# a cross of layer 2, and later operators that read such a cross's list
MULTI_CROSS_SPEC = ("fbx 1\nfields 4\n"
                    "op s hash slot=0 seed=1 emit=1 field=0 multi=0\n"
                    "op m hash slot=1 seed=2 emit=1 field=1 multi=1\n"
                    "op n hash slot=2 seed=3 emit=0 field=3 multi=1\n"
                    "op u bucket slot=3 seed=4 emit=1 field=2 multi=0 bounds=0,1000000\n"
                    "op x1 cross slot=4 seed=5 emit=1 a=s b=m\n"
                    "op x2 cross slot=5 seed=6 emit=1 a=m b=s\n"
                    "op x3 cross slot=6 seed=7 emit=0 a=u b=n\n"
                    "op x4 cross slot=7 seed=8 emit=1 a=s b=u\n"
                    "op x5 cross slot=8 seed=9 emit=1 a=x4 b=m\n"
                    "op x6 cross slot=9 seed=10 emit=1 a=x3 b=m\n"
                    "op x7 concat slot=10 emit=1 a=x1 b=x2\n"
                    "op x8 cross slot=11 seed=11 emit=1 a=m b=m\n"
                    "op x9 cross slot=12 seed=12 emit=1 a=n b=x4\n")


@pytest.mark.parametrize("mode", [{}, {"one_launch": 0}, {"fused": 0}] + TILE_MODES,
                         ids=["default", "two_launches", "per_layer"] + TILE_IDS)
def test_crosses_of_multi_valued_hashes_with_single_signs(mode):
    rng = random.Random(77)
    word = lambda: "".join(rng.choice("abcxyz0189") for _ in range(rng.randint(0, 9)))
    recs = []
    for i in range(333):
        items = lambda k: ",".join(word() for _ in range(k))
        k1 = rng.choice([1, 1, 2, 3, 5, 8, 16, 17, 21, 40])  # beyond the sixteen kept comma positions too
        k3 = rng.choice([1, 2, 4, 19])
        rec = f"{word()}\t{items(k1)}\t{rng.randint(-5, 5)}.{rng.randint(0, 999)}\t{items(k3)}"
        if i % 7 == 3:
            rec = word()  # the list fields are missing: one empty item each
        recs.append((rec + ("\n" if i % 3 else "")).encode())
    check(MULTI_CROSS_SPEC, *_cat(recs), mode, label=f"multi-valued crosses {mode}")


# prefixes of every length up to eight bytes, the limit of what the kernel keeps in registers, and
# beyond it; a comma inside the prefix (an ordinary byte for a single-valued filter, never matched
# by a token of a multi-valued one); filters that feed later layers
def _filter_spec():
    lines = ["fbx 1", "fields 3"]
    slot = 0
    for plen in (0, 1, 2, 3, 4, 5, 7, 8, 9, 12):
        for multi, field in ((0, 0), (1, 1)):
            lines.append(f"op f{plen}_{multi} filter slot={slot} seed={100 + slot} emit=1 field={field} "
                         f"multi={multi} prefix={(b'abababababab'[:plen]).hex()}")
            slot += 1
    lines.append(f"op c0 filter slot={slot} seed=50 emit=1 field=0 multi=0 prefix={b'a,b'.hex()}")
    lines.append(f"op c1 filter slot={slot + 1} seed=51 emit=0 field=1 multi=1 prefix={b'a,b'.hex()}")
    lines.append(f"op h hash slot={slot + 2} seed=52 emit=1 field=2 multi=0")
    lines.append(f"op x cross slot={slot + 3} seed=53 emit=1 a=f2_1 b=h")
    lines.append(f"op y concat slot={slot + 4} emit=1 a=c1 b=f1_0")
    lines.append(f"op z cross slot={slot + 5} seed=54 emit=1 a=x b=f0_0")
    return "\n".join(lines) + "\n"


@pytest.mark.parametrize("mode", [{}, {"one_launch": 0}, {"fused": 0}] + TILE_MODES,
                         ids=["default", "two_launches", "per_layer"] + TILE_IDS)
def test_filters_with_short_and_long_prefixes(mode):
    rng = random.Random(4242)

    def token():
        n = rng.choice([0, 1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 13, 20])
        t = "abababababababababababab"[:n]
        if n and rng.random() < 0.4:   # a mismatch at a random position, the last one included
            k = rng.randrange(n)
            t = t[:k] + rng.choice("bax") + t[k + 1:]
        return t + (rng.choice(["", "b", "zz"]) if rng.random() < 0.3 else "")

    recs = []
    for i in range(300):
        single = rng.choice([token(), "a,b" + token(), "a," + token(), token() + "," + token()])
        items = ",".join(token() for _ in range(rng.choice([1, 1, 2, 3, 6, 18, 30])))
        rec = f"{single}\t{items}\tk{i % 5}"
        if i % 11 == 5:
            rec = single  # the list field is missing: one empty token
        recs.append((rec + ("\n" if i % 4 else "")).encode())
    # a record that does not fit the staged text is read in place
    recs.append(b"abab\t" + ",".join(token() for _ in range(9000)).encode() + b"\tk1\n")
    check(_filter_spec(), *_cat(recs), mode, label=f"filters {mode}")


@pytest.mark.parametrize("cfg,one_launch,compile_for_plan", [(5, True, 1), (5, True, 0), (2, False, 1), (3, True, 1), (4, False, 1)],
                         ids=["config5", "config5_generic_kernel", "config2", "config3", "config4"])
def test_full_size_workloads_every_sign(cfg, one_launch, compile_for_plan):
    """The benchmark configurations at their full sizes, run the way bench.py times them (kernels
    compiled for the plan; a first call that sizes the workspace, then a call that knows the
    ragged sizes): properties that hold for the whole result, a few windows of records as a quick
    check, and then every slot's values and offsets against the oracle, which runs over disjoint
    record ranges on all host cores, chunk by chunk.  The largest one also with the generic kernel
    (its full comparison is left to the compiled kernel's run: the windows and properties stay)."""
    import sys
    import torch

    w = W.get(cfg)
    d_raw, d_off = device_workload(w)
    R = w.n_records
    plan = B.Plan(w.spec)
    plan.set_option("compile", compile_for_plan)
    first_res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.03)
    res = plan.extract(d_raw, d_off)
    assert res.tile_launches == (1 if one_launch else 2), res.note
    assert "generic kernel" not in res.note and (plan.compiled()[0] >= 2) == bool(compile_for_plan), res.note
    assert res.n_records == R and res.n_values_total == first_res.n_values_total
    total = 0
    for s in res.slot_ids:
        slot = res.slots[s]
        total += slot.n_values
        if slot.offsets is None:
            assert slot.n_values == R * slot.fixed_arity
            continue
        offs = slot.offsets
        assert offs.numel() == R + 1 and int(offs[0]) == 0 and int(offs[R]) == slot.n_values, f"slot {s}"
        assert bool((offs[1:] >= offs[:-1]).all()), f"slot {s}: offsets decrease"
    assert total == res.n_values_total
    rng = np.random.default_rng(1000 + cfg)
    starts = [0, R - 5, 31, 63, R // 2 - 2] + [int(x) for x in rng.integers(0, R - 5, size=(35 if not compile_for_plan else 5))]
    for first in starts:
        check_window(w.spec, res, d_raw, d_off, first, 5, label=f"{w.name} full size")
    if compile_for_plan:
        said = [0]

        def progress(done, of):  # (a line per tenth of the records: a long, quiet step otherwise)
            if done * 10 // of > said[0]:
                said[0] = done * 10 // of
                print(f"[{w.name}] {done}/{of} records compared with the oracle", file=sys.stderr, flush=True)

        n, _ = check_every_sign(w.spec, res, d_raw, d_off, chunk_records=250_000, label=f"{w.name} full size", progress=progress)
        assert n == res.n_values_total
    plan.close()
    del ws
    torch.cuda.empty_cache()


@pytest.mark.parametrize("cfg,n,compile_for_plan,grid_limit",
                         [(5, 200_000, 0, 0), (5, 200_000, 1, 0), (3, 300_000, 0, 0), (3, 300_000, 1, 0),
                          (5, 60_000, 1, 8), (3, 100_000, 0, 8)],
                         ids=["config5_generic", "config5_compiled", "config3_generic", "config3_compiled",
                              "config5_compiled_8_workgroups", "config3_generic_8_workgroups"])
def test_one_launch_mode_with_more_tiles_than_workgroups(cfg, n, compile_for_plan, grid_limit):
    """The one-launch sequence where it is timed: far more tiles than workgroups run at the same
    time, so that every workgroup takes tile after tile (parked offsets, the hand-over of what the
    offset check found, the look-back moving past its first window of 64 tiles), and with a grid
    of only eight workgroups, each of which then takes hundreds of tiles.  A first call (counting +
    writing), then two calls that place by look-back, the workspace scrubbed in between; every
    sign of every slot against the oracle."""
    from gpu_harness import expand
    w = W.get(cfg, n)
    raw, off = w.generate()
    slots, slot_ids, total, malformed = extract_parallel(w.spec, raw, off)
    plan = B.Plan(w.spec)
    plan.set_option("compile", compile_for_plan)
    if grid_limit:
        plan.set_option("grid_limit", grid_limit)
    d_raw, d_off = to_device(raw, off)
    res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.05)
    tiles = -(-n // (32 if cfg == 5 else 64))
    assert tiles > 2 * 512                  # (at most two workgroups on each of 256 compute units run at a time)
    for call in range(3):
        if call:
            ws.fill_(0xA5)
            plan.set_workspace(ws)
            res = plan.extract(d_raw, d_off)
            assert res.tile_launches == 1, res.note
        else:
            assert res.tile_launches == 2, res.note
        assert "generic kernel" not in res.note, res.note
        assert res.n_values_total == total and res.n_malformed_numeric == malformed
        assert list(res.slot_ids) == list(slot_ids)
        for s in slot_ids:
            gv, go = expand(res.slots[s], n)
            ov, oo, arity = slots[s]
            assert res.slots[s].fixed_arity == arity
            assert np.array_equal(go, oo), f"{w.name} call {call} slot {s}: offsets differ"
            assert np.array_equal(gv, ov), f"{w.name} call {call} slot {s}: signs differ"
    assert (plan.compiled()[0] >= 2) == bool(compile_for_plan)
    plan.close()


@pytest.mark.parametrize("tile_log2,compile_for_plan,grid_limit", [(5, 0, 0), (6, 0, 8), (5, 1, 0)])
def test_one_launch_mode_with_rows_that_follow_other_rows(tile_log2, compile_for_plan, grid_limit):
    """Ragged operators whose count per record is a multiple of another ragged operator's plus a
    constant (a cross or a concat with a fixed-arity input, a concat of two such operators over the
    same one, operators over those) are placed from that operator's look-back result in the
    one-launch sequence; a cross of two lists is not.  A first call, then two that place by
    look-back, over many tiles, every sign against the oracle."""
    from gpu_harness import expand
    rng = random.Random(4242 + tile_log2)
    n = 20_000  # (hundreds of tiles: the look-back moves past its first window)
    word = lambda: "".join(rng.choice("abcdefg") for _ in range(rng.randint(0, 40)))
    recs = [("\t".join([word(), word(), ",".join(word() for _ in range(rng.randint(1, 6))),
                         ",".join(word() for _ in range(rng.randint(1, 3)))]) + "\n").encode() for _ in range(n)]
    spec = FOLLOW_SPEC
    raw, off = _cat(recs)
    raw = np.frombuffer(raw, np.uint8)
    want = O.extract(spec, raw, off)
    plan = B.Plan(spec)
    plan.set_option("tile_log2", tile_log2)
    plan.set_option("compile", compile_for_plan)
    if grid_limit:
        plan.set_option("grid_limit", grid_limit)
    d_raw, d_off = to_device(raw, off)
    res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.05)
    for call in range(3):
        if call:
            ws.fill_(0x5A)
            plan.set_workspace(ws)
            res = plan.extract(d_raw, d_off)
            assert res.tile_launches == 1, res.note
        assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"call {call}")
    plan.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 777])
def test_tile_boundaries(n):
    for cfg in (5, 2):
        w = W.get(cfg, n)
        raw, off = w.generate()
        check(w.spec, raw, off, label=f"{w.name} n={n}")


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8192, 12289])
def test_tile_counts_around_the_scan_segments(n):
    # the scan over tiles cuts a row into segments of 4 096 tiles: one-record tiles put the record
    # count right at, one short of and one past whole segments
    rng = random.Random(n)
    recs = [(",".join("ab"[:rng.randint(0, 2)] for _ in range(rng.randint(1, 3))) + "\tq" + ("\n" if i % 2 else "")).encode()
            for i in range(n)]
    spec = ("fbx 1\nfields 2\n"
            "op a hash slot=0 seed=1 emit=1 field=0 multi=1\n"
            "op b hash slot=1 seed=2 emit=1 field=1 multi=0\n"
            "op c cross slot=2 seed=3 emit=1 a=a b=b\n"
            "op d cross slot=3 seed=4 emit=1 a=a b=a\n")
    check(spec, *_cat(recs), {"tile_log2": 0, "one_launch": 0}, label=f"{n} tiles")


@pytest.mark.parametrize("misalign", [1, 7, 15])
def test_unaligned_raw_pointer_and_slack(misalign):
    w = W.get(1, 300)
    raw, off = w.generate()
    # a gap before the first record and unused bytes after the last one
    raw2 = np.concatenate([np.frombuffer(b"junk\tjunk\n", np.uint8), raw, np.frombuffer(b"\ttail", np.uint8)])
    check(w.spec, raw2, off + np.uint64(10), misalign=misalign)


def test_empty_batch_and_single_record():
    out, res, plan = run_gpu(FRAMING_SPEC, np.zeros(0, np.uint8), np.zeros(1, np.uint64))
    assert res.n_values_total == 0
    for s, (v, o) in out.items():
        assert v.size == 0 and o.tolist() == [0]
    plan.close()
    check(FRAMING_SPEC, *_cat([FRAMING_RECORDS[0]]))
    check(FRAMING_SPEC, *_cat([b""]))


def test_long_records_and_dense_tabs():
    rng = random.Random(5)
    long_field = bytes(rng.choice(b"abcxyz,0123") for _ in range(70000))
    recs = [b"k\t" + long_field + b"\t1.25,7\tquery text here\n",
            b"a\tb\tc\td\n",
            b"\t" * 5000 + b"\n",            # far more tabs than fields
            b"m\tx1,x2\t-3.5\tabcdef\n"] * 3
    raw, off = _cat(recs)
    res, _ = check(FRAMING_SPEC, raw, off)
    # dense tabs
    recs = [b"\t\t\t" * 300 + b"\n"] * 40 + [b"a\tb,c\t1\tdddd\n"] * 40
    check(FRAMING_SPEC, *_cat(recs))


def test_malformed_numerics_are_counted():
    spec = ("fbx 1\nfields 2\n"
            "op a bucket slot=0 seed=1 emit=1 field=0 multi=1 bounds=-1000000,0,1000000\n"
            "op b bucket slot=1 seed=2 emit=0 field=1 multi=0 bounds=\n")
    recs = [b"1,x,-,.,-.5,1.2.3,99999999999999999999999\t12x\n", b"\t\n", b"-0.0000009,5\t7\n"] * 50
    res, want = check(spec, *_cat(recs))
    assert res.n_malformed_numeric == want.n_malformed_numeric > 0


def test_numeric_tokens_of_every_shape():
    """Numbers of every length and shape the grammar knows, and text that is not a number, as single
    values and as lists: short tokens take the kernel's loop-free conversion (a mask of non-digit
    bytes, four digits at a time), tokens beyond sixteen bytes and integer parts beyond eight digits
    its byte-by-byte fall-back; whatever follows a token in memory must not matter."""
    rng = random.Random(2024)
    digits = lambda k: "".join(rng.choice("0123456789") for _ in range(k))

    def token():
        kind = rng.random()
        if kind < 0.55:
            t = ("-" if rng.random() < 0.3 else "") + digits(rng.choice([0, 1, 1, 2, 3, 5, 8, 9, 12, 19, 23]))
            if rng.random() < 0.7:
                t += "." + digits(rng.choice([0, 1, 2, 5, 6, 7, 9, 14]))
            if rng.random() < 0.1:
                t += rng.choice(["x", ".", "-", "e5", " "])
            return t
        if kind < 0.8:
            return "".join(rng.choice("0123456789.-x") for _ in range(rng.choice([0, 1, 2, 3, 7, 8, 9, 15, 16, 17, 18, 30])))
        return rng.choice(["", "-", ".", "-.", "-.5", ".5", "1.", "00001.000001", "99999999", "999999999", "0.0000019",
                           "12345678.123456", "-12345678.1234567", "9" * 16, "9" * 17, "1" + "0" * 22])

    spec = ("fbx 1\nfields 3\n"
            "op a bucket slot=0 seed=1 emit=1 field=0 multi=0 bounds=-1000000,0,1,999999,1000000,12345678123456,99999999000000\n"
            "op b bucket slot=1 seed=2 emit=1 field=1 multi=1 bounds=-5000000,0,5000000\n"
            "op c bucket slot=2 seed=3 emit=1 field=2 multi=0 bounds=\n"
            "op x cross slot=3 seed=4 emit=1 a=a b=c\n")
    recs = [(f"{token()}\t{','.join(token().replace(',', '') for _ in range(rng.randint(1, 4)))}\t{token()}" + ("\n" if i % 2 else "")).encode()
            for i in range(20000)]
    for mode in ({}, {"compile": 1}, {"tile_log2": 6, "compile": 1, "lane_ops": 1}, {"fused": 0}):
        res, want = check(spec, *_cat(recs), mode, label=f"numeric tokens {mode}")
        assert res.n_malformed_numeric == want.n_malformed_numeric > 1000


def test_bad_offsets_are_rejected():
    w = W.get(1, 64)
    raw, off = w.generate()
    for mutate in ("decreasing", "beyond"):
        bad = off.copy()
        if mutate == "decreasing":
            bad[10] = bad[12]
        else:
            bad[-1] = raw.size + 5
        with pytest.raises(B.FbxError) as e:
            run_gpu(w.spec, raw, bad)
        assert e.value.status == B.E_INPUT


def test_more_signs_per_record_than_the_limit_is_an_input_error():
    """A cross of a list of 8200 items with itself would make 2^26 or more signs for one record:
    both launch sequences refuse the batch (and write nothing) instead of sizing arrays for it."""
    import torch
    spec = ("fbx 1\nfields 1\n"
            "op m hash slot=0 seed=1 emit=1 field=0 multi=1\n"
            "op x cross slot=1 seed=2 emit=1 a=m b=m\n")
    pad = b"0123456789abcdefghijklmnopqrstuvwxyz"  # (records long enough for the one-launch sequence to be chosen)
    small = [b"a" + pad + b",b,c" + pad + b"\n", b"d" + pad + pad + b"\n", pad + b"," + pad + b"\n", b"e,f" + pad + pad + b"\n"] * 30
    big = small[:50] + [b",".join([b"t"] * 8200) + b"\n"] + small[50:]
    def arrays(records):
        raw, off = _cat(records)
        return np.frombuffer(raw, np.uint8), off

    # first call on a plan: the counting launch sees it
    with pytest.raises(B.FbxError) as e:
        run_gpu(spec, *arrays(big))
    assert e.value.status == B.E_INPUT
    # a plan that knows its sizes from a good batch tries the one-launch sequence
    plan = B.Plan(spec)
    d_raw, d_off = to_device(*arrays(small))
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    plan.set_workspace(ws)
    plan.extract(d_raw, d_off)
    assert plan.extract(d_raw, d_off).tile_launches == 1
    d_raw2, d_off2 = to_device(*arrays(big))
    with pytest.raises(B.FbxError) as e:
        plan.extract(d_raw2, d_off2)
    assert e.value.status == B.E_INPUT
    # and the plan still works
    res = plan.extract(d_raw, d_off)
    want = O.extract(spec, *arrays(small))
    assert res.n_values_total == want.n_values_total
    plan.close()


def test_small_workspace_reports_requirement_then_succeeds():
    import torch
    w = W.get(2, 200)
    raw, off = w.generate()
    want = O.extract(w.spec, raw, off)
    plan = B.Plan(w.spec)
    d_raw, d_off = to_device(raw, off)
    hint = plan.workspace_hint(raw.size, 200)
    ws = torch.empty(262144, dtype=torch.uint8, device="cuda")
    plan.set_workspace(ws)
    with pytest.raises(B.FbxError) as e:
        plan.extract(d_raw, d_off)
    assert e.value.status == B.E_NOMEM and e.value.required_bytes > ws.numel()
    need = e.value.required_bytes
    for size, ok in ((need - 128, False), (need, True)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        plan.set_workspace(ws)
        if ok:
            res = plan.extract(d_raw, d_off)
            assert res.arena_high_water == need
            from gpu_harness import expand
            assert_same({s: expand(res.slots[s], 200) for s in res.slot_ids}, res, want)
        else:
            with pytest.raises(B.FbxError) as e2:
                plan.extract(d_raw, d_off)
            assert e2.value.status == B.E_NOMEM
    plan.close()


def test_repeated_calls_are_bit_identical_and_plan_is_reusable():
    w = W.get(4, 600)
    raw, off = w.generate()
    want = O.extract(w.spec, raw, off)
    plan = B.Plan(w.spec)
    d_raw, d_off = to_device(raw, off)
    res, ws = B.extract_with_retry(plan, d_raw, d_off)
    from gpu_harness import expand
    first = {s: expand(res.slots[s], 600) for s in res.slot_ids}
    assert_same(first, res, want)
    for k in range(10):
        if k % 2:
            ws.fill_(0x5A)      # stale results must not be able to stand in for missing writes
            plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)
        again = {s: expand(res.slots[s], 600) for s in res.slot_ids}
        for s in first:
            assert np.array_equal(first[s][0], again[s][0]) and np.array_equal(first[s][1], again[s][1])
    # a different, smaller batch on the same plan and workspace
    w2 = W.get(4, 100)
    raw2, off2 = w2.generate(rec_begin=5000, n_records=100)
    d_raw2, d_off2 = to_device(raw2, off2)
    res2 = plan.extract(d_raw2, d_off2)
    assert_same({s: expand(res2.slots[s], 100) for s in res2.slot_ids}, res2, O.extract(w.spec, raw2, off2))
    plan.close()


def test_one_launch_mode_matches_and_falls_back():
    # The second call on a plan sizes its ragged arrays from the first one and skips the
    # counting launch (bases by look-back between tiles); results must not change.  A batch
    # whose lists outgrow those arrays, or whose tiles need several passes, goes back to the
    # counting launch on its own.
    from gpu_harness import expand
    for cfg, n in ((5, 3000), (2, 400), (4, 900), (3, 2000)):
        w = W.get(cfg, n)
        raw, off = w.generate()
        want = O.extract(w.spec, raw, off)
        plan = B.Plan(w.spec)
        d_raw, d_off = to_device(raw, off)
        res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.2)
        assert res.tile_launches == (2 if any(s.offsets is not None for s in res.slots.values()) else 1)
        for _ in range(3):
            ws.fill_(0xAB)          # nothing an earlier call wrote may stand in for this call's results
            plan.set_workspace(ws)
            res = plan.extract(d_raw, d_off)
            # (plans with many ragged operators and short tiles keep the counting launch)
            assert res.tile_launches == (1 if cfg in (5, 3) else 2), w.name
            assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, w.name)
        # another batch of the same kind but a different size
        raw2, off2 = w.generate(rec_begin=10000, n_records=n // 3)
        d_raw2, d_off2 = to_device(raw2, off2)
        ws.fill_(0xCD)
        plan.set_workspace(ws)
        res2 = plan.extract(d_raw2, d_off2)
        assert res2.tile_launches == (1 if cfg in (5, 3) else 2), w.name
        assert_same({s: expand(res2.slots[s], n // 3) for s in res2.slot_ids}, res2, O.extract(w.spec, raw2, off2), w.name)
        plan.close()
    # lists that grow tenfold between calls: the arrays sized from the first call are too small
    spec = ("fbx 1\nfields 2\n"
            "op a hash slot=0 seed=1 emit=1 field=0 multi=1\n"
            "op b hash slot=1 seed=2 emit=1 field=1 multi=0\n"
            "op c cross slot=2 seed=3 emit=1 a=a b=b\n")
    pad = b"p" * 60   # (tiny records keep the counting launch: the placement words would outweigh them)
    short = [b"x\t" + pad + b"\n"] * 5000
    long_ = [b"a,b,c,d,e,f,g,h,i,j,k,l\t" + pad + b"\n"] * 5000
    plan = B.Plan(spec)
    import torch
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    plan.set_workspace(ws)
    for recs, launches in ((short, 2), (short, 1), (long_, 2), (long_, 1), (short, 1)):
        raw, off = _cat(recs)
        d_raw, d_off = to_device(np.frombuffer(raw, np.uint8), off)
        ws.fill_(0xEF)
        plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)
        assert res.tile_launches == launches
        assert_same({s: expand(res.slots[s], len(recs)) for s in res.slot_ids}, res, O.extract(spec, np.frombuffer(raw, np.uint8), off))
    # bad offsets in one-launch mode are still an error, and the plan keeps working afterwards
    raw, off = _cat(short)
    bad = off.copy(); bad[100] = bad[103]
    d_raw, d_off = to_device(np.frombuffer(raw, np.uint8), bad)
    with pytest.raises(B.FbxError) as e:
        plan.extract(d_raw, d_off)
    assert e.value.status == B.E_INPUT
    d_raw, d_off = to_device(np.frombuffer(raw, np.uint8), off)
    res = plan.extract(d_raw, d_off)
    assert_same({s: expand(res.slots[s], len(short)) for s in res.slot_ids}, res, O.extract(spec, np.frombuffer(raw, np.uint8), off))
    plan.close()


@pytest.mark.parametrize("compile_for_plan", [0, 1], ids=["generic", "compiled"])
def test_a_wait_between_tiles_that_runs_out_falls_back(compile_for_plan):
    """The one-launch sequence bounds its waits for earlier tiles.  A limit of zero polls, set from
    the host, makes every such wait run out at once: all kernels still run to their end and write
    nothing, the call is answered by the counting sequence, says so, and the plan keeps working."""
    from gpu_harness import expand
    w = W.get(5, 4000)
    raw, off = w.generate()
    want = O.extract(w.spec, raw, off)
    plan = B.Plan(w.spec)
    plan.set_option("compile", compile_for_plan)
    d_raw, d_off = to_device(raw, off)
    res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.2)
    res = plan.extract(d_raw, d_off)
    assert res.tile_launches == 1 and "wait" not in res.note
    plan.set_option("spin_limit", 0)
    for _ in range(2):
        ws.fill_(0x3C)
        plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)
        assert res.tile_launches == 2 and "bounded wait" in res.note, res.note
        assert_same({s: expand(res.slots[s], 4000) for s in res.slot_ids}, res, want, "after a wait ran out")
    plan.set_option("spin_limit", 1 << 22)
    ws.fill_(0xC3)
    plan.set_workspace(ws)
    res = plan.extract(d_raw, d_off)
    assert res.tile_launches == 1 and "wait" not in res.note, res.note
    assert_same({s: expand(res.slots[s], 4000) for s in res.slot_ids}, res, want, "one launch again")
    plan.close()


@pytest.mark.parametrize("case", ["config5", "config4", "config2", "config3", "framing", "filters_T8_cap64"])
def test_kernels_compiled_for_the_plan_match(case):
    """Plan option compile=1: the tile kernel is compiled again at run time with the plan's numbers
    written in (the meta-kernel of Section 4).  Counting, writing and one-launch kernels, a second
    batch of another size on the same kernels, several passes per tile and records read in place."""
    from gpu_harness import expand
    opts = {"compile": 1}
    if case.startswith("config"):
        cfg = int(case[-1])
        w = W.get(cfg, {5: 3000, 4: 900, 2: 400, 3: 2000}[cfg])
        spec = w.spec
        raw, off = w.generate()
        raw2, off2 = w.generate(rec_begin=10000, n_records=w.n_records // 3)
    elif case == "framing":
        spec = FRAMING_SPEC
        raw, off = _cat(FRAMING_RECORDS * 29)
        raw2, off2 = _cat(FRAMING_RECORDS * 3)
    else:
        spec = _filter_spec()
        opts.update({"tile_log2": 3, "raw_cap": 64})
        rng = random.Random(99)
        tok = lambda: "abababab"[:rng.randint(0, 8)] + rng.choice(["", "x"])
        recs = [f"{tok()}\t{','.join(tok() for _ in range(rng.randint(1, 12)))}\tk{i % 3}\n".encode() for i in range(200)]
        raw, off = _cat(recs)
        raw2, off2 = _cat(recs[:37])
    raw, raw2 = (np.frombuffer(x, np.uint8) if isinstance(x, bytes) else x for x in (raw, raw2))
    plan = B.Plan(spec)
    for k, v in opts.items():
        plan.set_option(k, v)
    d_raw, d_off = to_device(raw, off)
    res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.2)
    assert "generic kernel" not in res.note, res.note
    n_compiled = plan.compiled()[0]
    assert n_compiled >= 1                                   # (not the generic kernel under another name)
    n = len(off) - 1
    want = O.extract(spec, raw, off)
    assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, case)
    for _ in range(2):   # the calls after the first know the ragged sizes: one launch where the plan allows it
        ws.fill_(0xAB)
        plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)
        assert "generic kernel" not in res.note, res.note
        assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, case)
    d_raw2, d_off2 = to_device(raw2, off2)
    ws.fill_(0xCD)
    plan.set_workspace(ws)
    res2 = plan.extract(d_raw2, d_off2)
    assert "generic kernel" not in res2.note, res2.note
    assert_same({s: expand(res2.slots[s], len(off2) - 1) for s in res2.slot_ids}, res2, O.extract(spec, raw2, off2), case)
    assert n_compiled <= plan.compiled()[0] <= 6             # a kernel per mode and tile shape (the batch size may change the shape)
    plan.close()


@pytest.mark.parametrize("lane_ops,threads", [(1, 512), (2, 512), (1, 1024), (2, 1024)],
                         ids=["table_512", "generated_512", "table_1024", "generated_1024"])
def test_one_operator_per_wavefront_on_tiles_of_64_records(lane_ops, threads):
    """Kernels compiled for the plan, tiles of 64 records: a wavefront runs one single-sign operator at
    a time, one record per lane, its numbers read from the program table (lane_ops=1) or written
    into straight-line code generated for the plan, one case per operator (lane_ops=2: the
    meta-kernel of Section 4 in its own form); workgroups of 512 and of 1024 lanes.  Counting,
    writing and one-launch kernels, a ragged tail, a second batch, records read in place."""
    from gpu_harness import expand
    rng = random.Random(31)
    long_rec = b"k\t" + bytes(rng.choice(b"abcxyz,0123") for _ in range(70000)) + b"\t1.25,7\tquery text here\n"
    cases = [(W.get(5, 2500).spec, *W.get(5, 2500).generate()), (W.get(3, 3000).spec, *W.get(3, 3000).generate()),
             (W.get(1, 700).spec, *W.get(1, 700).generate()), (W.get(4, 500).spec, *W.get(4, 500).generate()),
             (FRAMING_SPEC, *_cat(FRAMING_RECORDS * 29 + [long_rec]))]
    for spec, raw, off in cases:
        raw = np.frombuffer(raw, np.uint8) if isinstance(raw, bytes) else raw
        n = len(off) - 1
        want = O.extract(spec, raw, off)
        plan = B.Plan(spec)
        for k, v in {"compile": 1, "tile_log2": 6, "lds_budget": 160 * 1024, "tile_threads": threads, "lane_ops": lane_ops}.items():
            plan.set_option(k, v)
        d_raw, d_off = to_device(raw, off)
        res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.2)
        assert "generic kernel" not in res.note, res.note
        assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"lane_ops={lane_ops} first call")
        for _ in range(2):
            ws.fill_(0xB7)
            plan.set_workspace(ws)
            res = plan.extract(d_raw, d_off)
            assert "generic kernel" not in res.note, res.note
            assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"lane_ops={lane_ops} later call")
        if not res.tile_launches:       # (a plan too wide for tiles of 64 records runs on the walk kernels)
            plan.close()
            continue
        assert plan.compiled()[0] >= 1
        src = plan.kernel_source(raw.size, n, 1)
        assert f"#define FBX_LANE_OPS {lane_ops}" in src and f"#define FBX_TILE_THREADS {threads}" in src
        assert ("lane_hash1(" in src or "lane_bucket1(" in src) == (lane_ops == 2)
        plan.close()


def _random_records(rng, n):
    def field():
        kind = rng.randrange(4)
        if kind == 0:
            return ",".join("abcab"[:rng.randint(0, 4)] for _ in range(rng.randint(1, 3)))
        if kind == 1:
            return ",".join(f"{rng.randint(-120, 120)}.{rng.randint(0, 99)}" for _ in range(rng.randint(1, 2)))
        if kind == 2:
            return "".join(rng.choice("abc .") for _ in range(rng.randint(0, 14)))
        return ""
    return [("\t".join(field() for _ in range(rng.randint(1, 5))) + ("\n" if i % 3 else "")).encode() for i in range(n)]


@pytest.mark.parametrize("seed", range(10))
def test_random_dags_against_the_oracle(seed):
    """Operator DAGs drawn at random (every kind of root on any field, crosses and concats of anything
    earlier, emitted or not), on records whose fields are lists, numbers, text or missing: generic and
    compiled kernels, one- and two-launch sequences, whole tiles and tiles in several passes."""
    from gpu_harness import expand
    rng = random.Random(1000 + seed)
    while True:
        spec, ids, deps = random_dag(rng, rng.randrange(2, 9), rng.randrange(1, 9))
        recs = _random_records(rng, rng.choice([70, 257, 600]))
        raw, off = _cat(recs)
        raw = np.frombuffer(raw, np.uint8)
        try:
            want = O.extract(spec, raw, off)
        except O.OracleError:
            continue                       # (a cross of crosses that outgrows the sign limit: draw again)
        if want.n_values_total <= 3_000_000:
            break
    modes = [{}, {"compile": 1}, {"tile_log2": 3, "raw_cap": 64}] if seed % 2 else [{}, {"one_launch": 0, "tile_log2": 5}]
    for mode in modes:
        plan = B.Plan(spec)
        for k, v in mode.items():
            plan.set_option(k, v)
        d_raw, d_off = to_device(raw, off)
        res, ws = B.extract_with_retry(plan, d_raw, d_off, slack=1.2)
        assert_same({s: expand(res.slots[s], len(recs)) for s in res.slot_ids}, res, want, f"seed {seed} {mode}")
        ws.fill_(0x5A)
        plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)   # the second call knows the sizes
        assert "generic kernel" not in res.note, res.note
        assert_same({s: expand(res.slots[s], len(recs)) for s in res.slot_ids}, res, want, f"seed {seed} {mode} again")
        plan.close()


def test_results_do_not_depend_on_op_order_or_launch_mode():
    w = W.get(4, 300)
    raw, off = w.generate()
    lines = w.spec.strip().split("\n")
    head, ops = lines[:2], lines[2:]
    roots = [l for l in ops if " cross " not in l and " concat " not in l]
    rest = [l for l in ops if l not in roots]
    random.Random(3).shuffle(roots)                # any order of the roots is topologically valid
    spec2 = "\n".join(head + roots + rest) + "\n"
    a, ra, pa = run_gpu(w.spec, raw, off, {"fused": 0})
    b, rb, pb = run_gpu(spec2, raw, off, {"fused": 1})
    assert sorted(a) == sorted(b)
    for s in a:
        assert np.array_equal(a[s][0], b[s][0]) and np.array_equal(a[s][1], b[s][1])
    pa.close(); pb.close()


def test_arena_reuse_lowers_the_high_water_mark():
    # non-emitted intermediates of early layers are released for later layers
    w = W.get(4, 2000)
    raw, off = w.generate()
    _, r_layered, p1 = run_gpu(w.spec, raw, off, {"fused": 0})
    _, r_fused, p2 = run_gpu(w.spec, raw, off, {"fused": 1})
    assert r_layered.arena_high_water <= r_fused.arena_high_water
    p1.close(); p2.close()


def test_algorithm1_arena_primitive():
    # Section 5, Algorithm 1: per-thread regions are disjoint, contiguous inside a
    # workgroup, sum to the bump of the head; workgroup bases are 128-byte aligned;
    # a reset makes the next allocation start from the pool base again.
    import torch
    rng = np.random.default_rng(9)
    for threads, n in ((64, 1000), (256, 5000), (1024, 3000)):
        sizes = rng.integers(0, 300, size=n).astype(np.int64)
        d_sizes = torch.from_numpy(sizes).cuda()
        d_off = torch.zeros(n, dtype=torch.int64, device="cuda")
        d_head = torch.tensor([4096], dtype=torch.int64, device="cuda")
        B.arena_alloc(d_head, d_sizes, d_off, threads)
        torch.cuda.synchronize()
        offs = d_off.cpu().numpy()
        head = int(d_head.cpu()[0])
        total = 0
        bases = []
        for b0 in range(0, n, threads):
            s, o = sizes[b0:b0 + threads], offs[b0:b0 + threads]
            assert o[0] % 128 == 0
            assert np.array_equal(o - o[0], np.cumsum(s) - s)      # exclusive prefix inside the workgroup
            bases.append((o[0], (int(s.sum()) + 127) // 128 * 128))
            total += bases[-1][1]
        assert head == 4096 + total
        bases.sort()
        assert bases[0][0] == 4096
        for (b, sz), (nb, _) in zip(bases, bases[1:]):
            assert b + sz == nb                                     # workgroup regions tile the bumped range
        B.arena_reset(d_head, 4096)
        B.arena_alloc(d_head, d_sizes[:threads], d_off[:threads], threads)
        torch.cuda.synchronize()
        assert int(d_off[0].cpu()) == 4096


def test_batches_with_a_tile_that_does_not_fit_stop_trying_the_one_launch_sequence():
    """One long record among short ones: its tile's text does not fit the LDS section, the one-launch attempt falls
    back, and the next call does not try again (then one more attempt, then two calls of rest, ...).  A batch
    without such a record takes one launch again once the rest is over.  Every call's result is the oracle's."""
    from gpu_harness import expand
    spec = ("fbx 1\nfields 2\n"
            "op a hash slot=0 seed=1 emit=1 field=0 multi=1\n"
            "op b hash slot=1 seed=2 emit=1 field=1 multi=0\n"
            "op c cross slot=2 seed=3 emit=1 a=b b=a\n")
    short = [b"xxxxxxxx,yyyyyyyy,zzzzzzzz\tqqqqqqqqqqqq\n"] * 3000   # (long enough for the one-launch sequence to be worth trying)
    with_long = list(short)
    with_long[1234] = b",".join([b"item"] * 30000) + b"\tq\n"   # 150 KB: more than any LDS section
    cat = lambda recs: (np.frombuffer(b"".join(recs), np.uint8), np.cumsum([0] + [len(r) for r in recs]).astype(np.uint64))
    want_long, want_short = O.extract(spec, *cat(with_long)), O.extract(spec, *cat(short))
    plan = B.Plan(spec)
    d_long, d_short = to_device(*cat(with_long)), to_device(*cat(short))
    res, ws = B.extract_with_retry(plan, *d_long, slack=1.2)
    seen = []
    for call in range(6):
        res = plan.extract(*d_long)
        assert res.tile_launches == 2
        seen.append("fell back" if "fell back" in res.note else ("rest" if "not tried" in res.note else res.note))
        assert_same({s: expand(res.slots[s], 3000) for s in res.slot_ids}, res, want_long, f"call {call}")
    assert seen == ["fell back", "rest", "fell back", "rest", "rest", "fell back"], seen
    for call in range(4):     # (four calls of rest are due)
        res = plan.extract(*d_short)
        assert res.tile_launches == 2 and "not tried" in res.note
    res = plan.extract(*d_short)
    assert res.tile_launches == 1, res.note
    assert_same({s: expand(res.slots[s], 3000) for s in res.slot_ids}, res, want_short, "short batch, one launch")
    res = plan.extract(*d_long)
    assert "fell back" in res.note   # (after a call that went through, the rests start over at one call)
    res = plan.extract(*d_long)
    assert "not tried" in res.note
    res = plan.extract(*d_long)
    assert "fell back" in res.note
    plan.close()


def test_plans_with_different_lds_sections_take_turns():
    """The kernel for any plan is one function: what one plan asks of it must not be in another one's way."""
    w = W.get(5, 300)
    raw, off = w.generate()
    want = O.extract(w.spec, raw, off)
    d_raw, d_off = to_device(raw, off)
    plans = []
    for cap in (60000, 8000, 60000):  # (sections of more than 64 KB with the tables, and of less)
        plan = B.Plan(w.spec)
        plan.set_option("tile_log2", 5)
        plan.set_option("raw_cap", cap)
        plan.set_option("one_launch", 0)
        plans.append(plan)
        B.extract_with_retry(plan, d_raw, d_off)
    for plan in plans + plans[::-1]:
        res = plan.extract(d_raw, d_off)
        assert_same({s: expand(res.slots[s], 300) for s in res.slot_ids}, res, want)
    for plan in plans:
        plan.close()


@pytest.mark.parametrize("lists,others,pad,commas", [
    (3, 0, 0, 0),      # hashes only: field by field
    (3, 4, 0, 1),      # filters and buckets of lists as well
    (3, 4, 3000, 2),   # the same on records of 3 KB: along with the tabs
    (40, 0, 0, 2),     # many lists: along with the tabs
])
@pytest.mark.parametrize("options", [{}, {"one_launch": 0}, {"placement": 1}, {"compile": 1}], ids=["default", "counting", "arrival", "compiled"])
def test_lists_around_the_commas_that_are_kept(lists, others, pad, commas, options):
    """Lists of up to 16 commas have all their places kept; longer ones, and records with more commas than their table holds
    (in fields that nobody reads as lists, too), are walked on from the last place."""
    rng = random.Random(lists * 100 + others)
    F = lists + others + 2
    spec = f"fbx 1\nfields {F}\nop t hash slot=900 seed=1 emit=1 field=0 multi=0\n"
    spec += "".join(f"op h{k} hash slot={k} seed={k} emit=1 field={1 + k} multi=1\n" for k in range(lists))
    for k in range(others):
        spec += (f"op o{k} filter slot={100 + k} seed={k} emit=1 field={1 + lists + k} multi=1 prefix={b'ab'[:k % 3].hex()}\n" if k % 2 == 0 else
                 f"op o{k} bucket slot={100 + k} seed={k} emit=1 field={1 + lists + k} multi=1 bounds=1000000,5000000\n")
    spec += "op x cross slot=901 seed=5 emit=1 a=h0 b=h1\nop y cross slot=902 seed=6 emit=1 a=t b=h2\n"
    recs = []
    for i in range(450):
        few = lambda: rng.choice([0, 1, 3, 3, 5]) if rng.random() < 0.9 else rng.choice([15, 16, 17, 18, 33, 60])
        items = lambda n: ",".join(rng.choice(["", "a", "ab", "abc7", "5.25", "x" * 20]) for _ in range(n + 1))
        text = "".join(rng.choice("ab,") for _ in range(rng.choice([0, 10, 700] if i % 5 == 0 else [0, 8])))
        fields = [text] + [items(few()) for _ in range(lists + others)] + ["z" * (pad + rng.randrange(20))]
        recs.append(("\t".join(fields) + "\n").encode())
    raw, off = _cat(recs)
    raw = np.frombuffer(raw, np.uint8)
    want = O.extract(spec, raw, off)
    plan = B.Plan(spec)
    for k, v in options.items():
        if k != "placement":
            plan.set_option(k, v)
    assert f"P.commas = {commas}u;" in plan.kernel_source(raw.size, 450, 1)
    d_raw, d_off = to_device(raw, off, 3)
    B.extract_with_retry(plan, d_raw, d_off)
    for k, v in options.items():
        if k == "placement":
            plan.set_option(k, v)
    for _ in range(2):
        res = plan.extract(d_raw, d_off)
        if "placement" in options:
            assert res.n_values_total == want.n_values_total and res.n_malformed_numeric == want.n_malformed_numeric
            continue
        assert_same({s: expand(res.slots[s], 450) for s in res.slot_ids}, res, want)
    plan.close()


@pytest.mark.parametrize("n_ops", [63, 64, 65, 255, 256, 257, 879, 880, 881, 1500])
def test_plans_of_many_operators(n_ops):
    """Placements travel with the set-up launch in blocks of 64, 256 and 880, or in memory beyond that."""
    rng = random.Random(n_ops)
    spec = "fbx 1\nfields 5\n" + "".join(f"op h{k} hash slot={k} seed={rng.getrandbits(64)} emit=1 field={k % 5} multi=0\n" for k in range(n_ops))
    raw, off = _cat([("\t".join("abc"[:rng.randrange(4)] for _ in range(5)) + "\n").encode() for _ in range(130)])
    check(spec, raw, off, label=str(n_ops))


@pytest.mark.parametrize("n_lists", [31, 32, 127, 129, 439, 441])
def test_plans_of_many_list_operators(n_lists):
    """The same where every operator has an offsets array of its own: two placements an operator, made on the host in the
    second call (a batch of one tile, whose arrival order is the records')."""
    import torch
    rng = random.Random(n_lists)
    spec = "fbx 1\nfields 5\n" + "".join(f"op h{k} hash slot={k} seed={rng.getrandbits(64)} emit=1 field={k % 5} multi=1\n" for k in range(n_lists))
    raw, off = _cat([("\t".join("a,bc,,d"[:rng.randrange(8)] for _ in range(5)) + "\n").encode() for _ in range(4)])
    raw = np.frombuffer(raw, np.uint8)
    want = O.extract(spec, raw, off)
    plan = B.Plan(spec)
    plan.set_option("placement", 1)
    plan.set_option("tile_log2", 2)
    d_raw, d_off = to_device(raw, off)
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    plan.set_workspace(ws)
    plan.extract(d_raw, d_off)
    res = plan.extract(d_raw, d_off)
    assert res.tile_launches == 1 and 4 == res.arrival_tile_records, res.note
    assert_same({s: expand(res.slots[s], 4) for s in res.slot_ids}, res, want)
    plan.close()


@pytest.mark.parametrize("crosses", [63, 64, 65, 150])
@pytest.mark.parametrize("tile_log2", [2, 5])
def test_layers_of_many_list_crosses(crosses, tile_log2):
    """Up to 64 list operators of a layer are found with one look by a wavefront, more by a search (and records by either)."""
    rng = random.Random(crosses)
    spec = "fbx 1\nfields 6\n" + "".join(f"op h{k} hash slot={k} seed={k} emit=1 field={k} multi=1\n" for k in range(6))
    spec += "".join(f"op x{k} cross slot={100 + k} seed={rng.getrandbits(64)} emit=1 a=h{rng.randrange(6)} b=h{rng.randrange(6)}\n" for k in range(crosses))
    raw, off = _cat([("\t".join(rng.choice(["a", "a,bc", ",,d", "q,w,e,r"]) for _ in range(6)) + "\n").encode() for _ in range(101)])
    for compiled in (0, 1):
        check(spec, raw, off, {"tile_log2": tile_log2, "compile": compiled}, label=f"{crosses} {tile_log2} {compiled}")


LISTS_ON_CHIP_SPEC = ("fbx 1\nfields 5\n"
                      "op s hash slot=0 seed=1 emit=0 field=0 multi=0\n"
                      "op m hash slot=1 seed=2 emit=0 field=1 multi=1\n"
                      "op n hash slot=2 seed=3 emit=1 field=2 multi=1\n"
                      "op b bucket slot=3 seed=4 emit=0 field=3 multi=1 bounds=0,2000000\n"
                      "op f filter slot=4 seed=5 emit=0 field=2 multi=1 prefix=61\n"
                      "op g ngram slot=5 seed=6 emit=0 field=4 n=3\n"
                      "op c concat slot=6 emit=0 a=s b=s\n"
                      "op k cross slot=7 seed=7 emit=0 a=s b=m\n"
                      "op x cross slot=8 seed=8 emit=0 a=m b=n\n"
                      "op y cross slot=9 seed=9 emit=1 a=b b=f\n"
                      "op z concat slot=10 emit=0 a=g b=m\n"
                      "op d cross slot=11 seed=10 emit=1 a=c b=n\n"
                      "op e concat slot=12 emit=1 a=c b=c\n"
                      "op w concat slot=13 emit=0 a=x b=z\n"
                      "op q cross slot=14 seed=11 emit=0 a=k b=f\n"
                      "op r concat slot=15 emit=1 a=w b=q\n"
                      "op t cross slot=16 seed=12 emit=1 a=q b=c\n")


@pytest.mark.parametrize("most", [3, 30])
@pytest.mark.parametrize("options", [{}, {"one_launch": 0}, {"compile": 1}, {"tile_log2": 0}, {"tile_log2": 5, "raw_cap": 1024},
                                     {"tile_log2": 4, "raw_cap": 1024, "compile": 1}, {"lds_budget": 20000}])
def test_lists_that_stay_on_chip(options, most):
    """Lists that later operators read (of every kind of operator, emitted or not) where all, some or none of them find room
    on chip, in tiles of one pass and of several, and of records that are read in place."""
    rng = random.Random(most)
    word = lambda: "".join(rng.choice("abc019") for _ in range(rng.randint(0, 6)))
    items = lambda make: ",".join(make() for _ in range(rng.randint(1, most)))
    recs = []
    for i in range(150):
        rec = "\t".join([word(), items(word), items(word), items(lambda: f"{rng.randint(-3, 9)}.{rng.randint(0, 9)}"), word() * rng.randint(0, 9)])
        recs.append((word() if i % 11 == 3 else rec * (40 if i % 50 == 7 else 1)).encode() + b"\n")
    check(LISTS_ON_CHIP_SPEC, *_cat(recs), options, label=f"{options} {most}")


@pytest.mark.parametrize("options", [{}, {"compile": 1}, {"fused": 0}])
def test_concats_of_single_signs_without_any_list(options):
    spec = ("fbx 1\nfields 2\nop a hash slot=0 seed=1 emit=0 field=0 multi=0\nop b hash slot=1 seed=2 emit=1 field=1 multi=0\n"
            "op c concat slot=2 emit=1 a=a b=b\nop d cross slot=3 seed=3 emit=1 a=c b=a\n")
    raw, off = _cat([f"{i}\tx{i * i}\n".encode() for i in range(333)])
    check(spec, raw, off, options, label=str(options))


@pytest.mark.parametrize("cfg,n", [(1, 1), (1, 65), (1, 513), (5, 1), (5, 5), (5, 255), (5, 256), (5, 257), (5, 513), (5, 1025), (2, 9), (2, 257), (2, 700),
                                   (3, 257), (3, 2048), (3, 2049), (4, 65), (4, 300)])
def test_batches_of_few_tiles(cfg, n):
    """Tiles are halved while a batch has few of them: sizes around the steps, in the call that counts and in the ones that look
    back, with a workspace that has room for their tables and with one that only has room for those of whole tiles."""
    import torch
    w = W.get(cfg, n)
    raw, off = w.generate()
    want = O.extract(w.spec, raw, off)
    d_raw, d_off = to_device(raw, off)
    plan = B.Plan(w.spec)
    res, ws = B.extract_with_retry(plan, d_raw, d_off)
    for _ in range(2):
        res = plan.extract(d_raw, d_off)
        assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"config{cfg} {n}")
    plan.close()
    plan = B.Plan(w.spec)
    size = 512 << 10
    for _ in range(5):  # (what is asked for when a call is refused has to be enough in the end, and stay enough)
        plan.set_workspace(torch.empty(size, dtype=torch.uint8, device="cuda"))
        try:
            for call in range(3):
                res = plan.extract(d_raw, d_off)
                assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"config{cfg} {n}, tight, call {call}")
            break
        except B.FbxError as e:
            assert e.status == B.E_NOMEM and e.required_bytes > size
            size = e.required_bytes
    else:
        pytest.fail(f"a workspace of {size} bytes is refused, as were the ones asked for before it")
    plan.close()


@pytest.mark.parametrize("cfg,n,fewer", [(5, 257, 100), (5, 1000, 300), (3, 2000, 700)])
def test_workspaces_that_hold_the_tables_of_whole_tiles_only(cfg, n, fewer):
    """Smaller tiles have larger tables.  A workspace without room for those takes whole tiles, in the call that counts and in
    one sized from the last call's signs; one that is too small either way is told what whole tiles need, and batches of
    fewer records still take smaller tiles in it."""
    import re

    import torch
    w = W.get(cfg, n)
    raw, off = w.generate()
    d_raw, d_off = to_device(raw, off)
    batch = {m: (d_raw[:int(off[m])], d_off[:m + 1], O.extract(w.spec, raw[:int(off[m])], off[:m + 1])) for m in (n, fewer)}

    def plan_with(size, tile_log2=-1):
        plan = B.Plan(w.spec)
        plan.set_option("tile_log2", tile_log2)
        plan.set_workspace(torch.empty(size, dtype=torch.uint8, device="cuda"))
        return plan

    def call(plan, m):
        d, o, want = batch[m]
        res = plan.extract(d, o)
        assert_same({s: expand(res.slots[s], m) for s in res.slot_ids}, res, want, f"config{cfg} {m}")
        return res.arena_high_water, res.tile_launches

    log2 = int(re.search(r"P\.log2T = (\d+)u;", B.Plan(w.spec).kernel_source(raw.size, n, 1)).group(1))
    room = 256 << 20
    plan = plan_with(room)
    (split, _), (split_margin, _) = call(plan, n), call(plan, n)
    plan = plan_with(room, log2)
    (whole, _), (whole_margin, _) = call(plan, n), call(plan, n)
    fewer_split, _ = call(plan_with(room), fewer)
    assert whole < min(split, whole_margin) and max(split, whole_margin) < split_margin

    assert call(plan_with(whole), n) == (whole, 2)
    for size in (split, whole_margin):
        plan = plan_with(size)
        first = (split if split <= size else whole, 2)
        then = (whole_margin, 1) if whole_margin <= size else first
        assert [call(plan, n) for _ in range(3)] == [first, then, then]
    plan = plan_with(whole - 128)
    with pytest.raises(B.FbxError) as e:
        call(plan, n)
    assert e.value.status == B.E_NOMEM and e.value.required_bytes == whole
    assert call(plan, fewer) == (fewer_split, 2)


@pytest.mark.parametrize("n", range(1, 9))
@pytest.mark.parametrize("options", [{}, {"compile": 1}, {"tile_log2": 5, "raw_cap": 1024}])
def test_ngrams_that_later_operators_read(options, n):
    """Grams of one word and of two, of fields shorter than a gram, of exactly one, of a wavefront's lanes and of one more, where all,
    some or none of the lists stay on chip, at every place of a word."""
    spec = (f"fbx 1\nfields 3\nop a ngram slot=0 seed=1 emit=1 field=0 n={n}\nop b ngram slot=1 seed=2 emit=0 field=2 n={n}\n"
            f"op c ngram slot=2 seed=3 emit=1 field=1 n={n}\nop d concat slot=3 emit=1 a=a b=b\nop e cross slot=4 seed=4 emit=1 a=c b=b\n")
    rng = random.Random(n)
    text = lambda k: "".join(rng.choice("abcdef,") for _ in range(k))
    recs = []
    for i in range(130):
        k = rng.choice([0, 1, n - 1, n, n + 1, 20, 62 + n, 63 + n, 64 + n, 128 + n])
        recs.append(f"{text(k)}\t{text(i % 7 + n - 1)}\t{text(rng.choice([n - 1, n, n + 3]))}\n".encode())
    check(spec, *_cat(recs), options, label=f"{options} {n}")


@pytest.mark.parametrize("pad,long_tokens", [(0, 0), (40, 1)])
def test_tokens_of_every_length_in_kernels_compiled_for_short_and_long_ones(pad, long_tokens):
    """Tokens of no bytes to five windows of eight, each at every place of a word, beside ones of other lengths."""
    spec = ("fbx 1\nfields 4\nop a hash slot=0 seed=1 emit=1 field=0 multi=0\nop b hash slot=1 seed=2 emit=1 field=1 multi=1\n"
            "op c filter slot=2 seed=3 emit=1 field=1 multi=1 prefix=61\nop d hash slot=3 seed=4 emit=1 field=2 multi=0\n"
            "op x cross slot=4 seed=5 emit=1 a=b b=c\n")
    rng = random.Random(pad)
    text = lambda k: "".join(rng.choice("abcdefgh") for _ in range(k))
    recs = []
    for i in range(410):
        items = ",".join(text(rng.choice([0, 1, 7, 8, 9, 12, 16, 17])) for _ in range(i % 3))
        recs.append(f"{text(i % 41 if i % 4 == 0 else i % 9)}\t{items}\t{text(rng.choice([0, 3, 8, 11, 12, 13]))}\t{text(pad)}\n".encode())
    raw, off = _cat(recs)
    plan = B.Plan(spec)
    plan.set_option("compile", 1)
    assert f"#define FBX_LONG_TOKENS {long_tokens}\n" in plan.kernel_source(len(raw), len(recs), 1)
    plan.close()
    check(spec, raw, off, {"compile": 1}, label=f"pad {pad}")


@pytest.mark.parametrize("options", [{"tile_log2": 0}, {"tile_log2": 3}, {"tile_log2": 6}, {"tile_log2": 4, "raw_cap": 1024}, {"tile_log2": 3, "compile": 1},
                                     {"tile_log2": 6, "one_launch": 0, "compile": 1}], ids=str)
@pytest.mark.parametrize("rare", [1, 70])
def test_list_operators_that_are_mostly_empty(rare, options):
    """Runs of (operator, record) pairs without signs, as long as several wavefronts, between pairs of a few signs and of more
    than a wavefront; layers of few and of more than 64 operators; fixed arities 2, 3 and 6 beside them."""
    rng = random.Random(rare)
    spec = "fbx 1\nfields 4\nop s hash slot=0 seed=1 emit=0 field=0 multi=0\nop m hash slot=1 seed=2 emit=0 field=1 multi=1\n"
    spec += "op q filter slot=2 seed=3 emit=0 field=2 multi=0 prefix=7a7a\n"
    spec += "".join(f"op r{k} cross slot={10 + k} seed={rng.getrandbits(64)} emit={k % 2} a={'qm'[k % 2]} b={'qmq'[k % 3]}\n" for k in range(rare))
    spec += "op c2 concat slot=3 emit=1 a=s b=s\nop c3 concat slot=4 emit=1 a=c2 b=s\nop x6 cross slot=5 seed=4 emit=1 a=c3 b=c2\n"
    spec += "op l concat slot=6 emit=1 a=q b=m\nop y cross slot=7 seed=5 emit=1 a=c3 b=l\nop z cross slot=8 seed=6 emit=1 a=r0 b=x6\n"
    recs = []
    for i in range(403):
        items = rng.choice([0, 1, 2]) if i % 40 else 90
        recs.append(("\t".join([f"t{i}", ",".join(rng.choice(["", "a", "bcd"]) for _ in range(items + 1)),
                                "zz9" if rng.random() < 0.02 else "y", "pad" * rng.randrange(5)]) + "\n").encode())
    raw, off = _cat(recs)
    check(spec, raw, off, options, label=f"{rare} {options}")


@pytest.mark.parametrize("compiled", [0, 1])
def test_what_counting_leaves_for_the_writing_launch(compiled):
    """Batches that count: what the counting launch found is taken over tile by tile, except for tiles with too many commas in
    a record or more signs of an operator than 16 bits hold, and for all of them where the workspace has no room for it or the
    arrays have grown into it.  Every size of workspace between what the arrays need and far beyond gives the same results."""
    import torch
    rng = random.Random(3)
    F = 16
    spec = f"fbx 1\nfields {F}\n" + "".join(f"op h{k} hash slot={k} seed={k} emit=1 field={k} multi=1\n" for k in range(12))
    spec += "op f filter slot=20 seed=7 emit=1 field=13 multi=1 prefix=61\nop s hash slot=21 seed=8 emit=1 field=14 multi=0\n"
    spec += "op x cross slot=22 seed=9 emit=1 a=h0 b=h1\nop y cross slot=23 seed=10 emit=1 a=x b=s\nop z concat slot=24 emit=1 a=f b=h2\n"
    def batch(n, dense):
        recs = []
        for i in range(n):
            many = {7: 300, 8: 90, 9: 17}.get(i % dense, 0)
            lists = [",".join(rng.choice(["a", "bb", "", "a" * 30]) for _ in range(rng.randrange(1, 5) + many)) for _ in range(14)]
            recs.append(("\t".join(lists + [f"k{i}", "t" * (1500 + rng.randrange(300))]) + "\n").encode())
        raw, off = _cat(recs)
        return np.frombuffer(raw, np.uint8), off
    for n, dense in ((331, 100), (40, 10)):
        raw, off = batch(n, dense)
        want = O.extract(spec, raw, off)
        d_raw, d_off = to_device(raw, off, 5)
        need = None
        for extra in (None, 0, 3000, 200_000, 1 << 20, 1 << 23):
            plan = B.Plan(spec)
            plan.set_option("one_launch", 0)
            plan.set_option("tile_log2", 3)
            plan.set_option("compile", compiled)
            assert "P.kept_bytes = 0u;" not in plan.kernel_source(raw.size, n, 1)
            if extra is None:
                res, ws = B.extract_with_retry(plan, d_raw, d_off)
                need = res.arena_high_water
            else:
                ws = torch.full((need + extra,), 0xff, dtype=torch.uint8, device="cuda")
                plan.set_workspace(ws)
                res = plan.extract(d_raw, d_off)
            for _ in range(2):
                assert res.tile_launches == 2, res.note
                assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"{n} {extra}")
                res = plan.extract(d_raw, d_off)
            plan.close()


@pytest.mark.parametrize("compiled", [0, 1])
@pytest.mark.parametrize("log2,pad", [(0, 2200), (3, 2200), (6, 200)])
def test_slots_of_the_counting_launch_are_taken_over_tile_by_tile(log2, pad, compiled):
    """The first word of a tile's slot says whether the writing launch takes it over: 1 for tiles worked off in one pass whose
    commas and signs a slot has room for, 0 for the others, and no slot is written where the workspace has no room for all."""
    import re

    import torch
    rng = random.Random(log2)
    n = {0: 37, 3: 203, 6: 403}[log2]  # (the last tile of 8 and of 64 records is not full)
    spec = "fbx 1\nfields 16\n" + "".join(f"op h{k} hash slot={k} seed={k} emit=1 field={k} multi=1\n" for k in range(12))
    spec += "op s hash slot=21 seed=8 emit=1 field=14 multi=0\nop x cross slot=22 seed=9 emit=1 a=h0 b=h1\nop y cross slot=23 seed=10 emit=1 a=x b=s\n"
    if log2 < 6:
        spec += "op f filter slot=20 seed=7 emit=1 field=13 multi=1 prefix=61\nop z concat slot=24 emit=1 a=f b=h2\n"
    recs = []
    for i in range(n):
        # (a record with more commas than a slot has room for; one with 270 * 270 signs of the cross; one beside the usual)
        many = {5: [200] * 3, n // 2: [270] * 2, n - 1: [9]}.get(i, [0])
        lists = [",".join(rng.choice(["a", "bb", "", "ccc"]) for _ in range(rng.randrange(1, 5) + (many[k] if k < len(many) else 0))) for k in range(14)]
        text = "t" * (pad + rng.randrange(pad // 5 + 1))
        if log2 == 6 and 256 <= i < 320:  # (more than 65,535 signs of the cross from lists that a slot has room for)
            lists, text = ["a" + ",a" * 35] * 2 + ["b"] * 12, ""
        recs.append(("\t".join(lists + [f"k{i}", text]) + "\n").encode())
    raw, off = _cat(recs)
    raw = np.frombuffer(raw, np.uint8)
    want = O.extract(spec, raw, off)
    d_raw, d_off = to_device(raw, off, 3)

    def plan_of():
        plan = B.Plan(spec)
        for k, v in (("one_launch", 0), ("tile_log2", log2), ("compile", compiled)):
            plan.set_option(k, v)
        return plan

    plan = plan_of()
    text = plan.kernel_source(raw.size, n, 1)
    field = {k: int(re.search(rf"P\.{k} = (\d+)u;", text).group(1)) for k in ("log2T", "commas", "raw_cap", "kept_bytes", "kept_commas")}
    assert field["log2T"] == log2 and field["commas"] == 2 and field["kept_bytes"]
    res, _ = B.extract_with_retry(plan, d_raw, d_off)
    need = res.arena_high_water
    plan.close()
    T = 1 << log2
    expected = []
    ragged = [want.slots[s][1] for s in want.slot_ids if want.slots[s][2] == 0]
    for t in range(0, n, T):
        e = min(t + T, n)
        delta = (d_raw.data_ptr() + int(off[t])) % 16
        fits = int(off[e]) - int(off[t]) + delta <= field["raw_cap"]
        commas = max(r.count(b",") for r in recs[t:e])
        signs = max(int(o[e]) - int(o[t]) for o in ragged)
        expected.append(1 if fits and commas <= field["kept_commas"] and signs <= 0xffff else 0)
        if t == 256 and log2 == 6:
            assert fits and commas <= field["kept_commas"] and signs > 0xffff
    assert 0 in expected and 1 in expected and (log2 == 6 or expected[-1] == 1)
    size = (len(expected) * field["kept_bytes"] + 255) // 256 * 256
    for extra in (size + 4096, (1 << 21) + size):
        plan = plan_of()
        ws = torch.full((need + extra,), 0xff, dtype=torch.uint8, device="cuda")
        plan.set_workspace(ws)
        res = plan.extract(d_raw, d_off)
        assert res.tile_launches == 2, res.note
        assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"{log2} {extra}")
        at = (need + extra - size) // 256 * 256
        words = ws[at:at + len(expected) * field["kept_bytes"]].view(len(expected), -1)[:, :4].contiguous().cpu().numpy().view(np.uint32)[:, 0]
        assert words.tolist() == expected
        plan.close()
    # a workspace of the size that the call needs, once the plan knows that: nothing is written behind the arrays
    plan = plan_of()
    plan.set_workspace(torch.empty(need + size + 4096, dtype=torch.uint8, device="cuda"))
    plan.extract(d_raw, d_off)
    ws = torch.full((need + 4096,), 0xff, dtype=torch.uint8, device="cuda")
    plan.set_workspace(ws)
    res = plan.extract(d_raw, d_off)
    assert_same({s: expand(res.slots[s], n) for s in res.slot_ids}, res, want, f"{log2} no room")
    assert bool((ws[need:] == 0xff).all())
    plan.close()
