"""Host-only checks of the C-ABI library: it loads, exports every symbol the header
declares, and its pure size arithmetic is right.  No compute call is made here."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mk():
    from paper_2512_22195_amd import LIB_PATH, build
    if not os.path.exists(LIB_PATH):
        build()
    from paper_2512_22195_amd import binding
    return binding


def test_library_exports_every_declared_symbol(mk):
    header = open(os.path.join(ROOT, "include", "matkv.h")).read()
    declared = set(re.findall(r"\b(matkv_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found in include/matkv.h"
    assert declared == set(mk.EXPORTS), declared ^ set(mk.EXPORTS)
    for name in declared:
        assert hasattr(mk.lib(), name), f"libmatkv.so does not export {name}"


def test_blob_bytes_formula_and_paper_orders_of_magnitude(mk):
    """n_layers * 2 * Hkv * n_tokens * D * 2 bytes.  The paper (Section II-C) quotes about
    100 MB per 1000 tokens for a 3B LLaMA and BASELINE's stream config about 1.3 GB for ten
    1000-token chunks of the 8B shape."""
    c8 = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, 1, 10, 192)
    assert mk.blob_bytes(c8, 1000) == 32 * 2 * 8 * 1000 * 128 * 2 == 131_072_000
    assert abs(10 * mk.blob_bytes(c8, 1000) / 1e9 - 1.3) < 0.02
    # 3B shape: 28 layers, 8 KV heads, D 128 (its 24 query heads, group 3, do not enter the size)
    c3 = mk.make_config(28, 8, 8, 128, 3072, "bf16", 500000.0, 1, 10, 192)
    mb = mk.blob_bytes(c3, 1000) / 1e6
    assert mb == pytest.approx(114.688) and 80 < mb < 130      # "approximately 100 MB"
    c70 = mk.make_config(80, 64, 8, 128, 8192, "bf16", 500000.0, 4, 20, 384)
    assert mk.blob_bytes(c70, 1000) == 327_680_000
    c1 = mk.make_config(1, 4, 2, 64, 256, "f32", 10000.0, 1, 2, 40)
    assert mk.blob_bytes(c1, 256) == 262_144
    assert mk.tail_bytes(c1) == 1 * 2 * 40 * 64 * 4
    assert mk.blob_bytes(c1, -1) == 0


def test_config_check_rejects_what_is_not_built(mk):
    ok = dict(n_layers=1, n_q_heads=4, n_kv_heads=2, head_dim=64, hidden=256, dtype="f32",
              rope_base=10000.0, max_batch=1, max_pages=2, max_tail_tokens=40)
    assert mk.config_check(mk.make_config(**ok)) == mk.OK
    bad = [dict(head_dim=96), dict(n_q_heads=6, n_kv_heads=4), dict(n_q_heads=32, n_kv_heads=2),
           dict(hidden=100), dict(max_tail_tokens=41), dict(n_layers=0), dict(rope_base=1.0),
           dict(decode_units=1000), dict(max_batch=0)]
    for delta in bad:
        cfg = mk.make_config(**{**ok, **delta})
        assert mk.config_check(cfg) in (mk.EINVAL, mk.EUNSUPPORTED), delta
        assert mk.workspace_bytes(cfg) == 0 and mk.table_bytes(cfg) == 0
    assert mk.config_check(mk.make_config(**{**ok, "head_dim": 96})) == mk.EUNSUPPORTED
    assert mk.lib().matkv_status_string(3) == b"MATKV_ENOTREADY"


def test_workspace_and_table_sizes_are_positive_and_aligned(mk):
    c = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, 16, 5, 192)
    assert mk.workspace_bytes(c) % 256 == 0 and mk.workspace_bytes(c) > 0
    assert mk.table_bytes(c) % 256 == 0 and mk.table_bytes(c) > 0
    # bf16 / head_dim 128: room for the projection's split tiles (128 tiles x two fp32 partials of
    # 128 x 128) however small the attention's own needs are
    small = mk.make_config(1, 8, 2, 128, 512, "bf16", 500000.0, 1, 1, 8)
    assert mk.workspace_bytes(small) >= 128 * 2 * 128 * 128 * 4
    # hidden 8192: tiles of up to 256 rows are split as well, whatever the longest tail and the head count
    for hq, max_tail in ((8, 8), (64, 16), (16, 64)):
        assert mk.workspace_bytes(mk.make_config(1, hq, 8, 128, 8192, "bf16", 500000.0, 1, 1, max_tail)) >= 128 * 2 * 256 * 128 * 4


def test_workspace_holds_no_more_than_the_split_tiles_leave(mk):
    """Tiles of 128 rows and more leave one partial each, lower ones two: up to hidden 8192, whose configurations split tiles of up to 192 rows, two
    of 128 rows hold either.  (Beside the partials: a page and a counter line of each tile.)"""
    for hidden in (512, 2048, 2560, 3072, 4096, 7168):
        small = mk.workspace_bytes(mk.make_config(1, 8, 2, 128, hidden, "bf16", 500000.0, 1, 1, 8))
        assert 128 * 192 * 128 * 4 <= small <= 128 * 2 * 128 * 128 * 4 + 8192 + 128 * 128


def test_null_context_is_an_error_not_a_crash(mk):
    assert mk.lib().matkv_destroy(None) == mk.EINVAL
    assert mk.lib().matkv_advance(None, None, 1) == mk.EINVAL
    assert mk.lib().matkv_last_error(None) == b"context is null"


def test_decode_partition_covers_every_token_once_and_is_balanced(mk):
    """Host logic of cache assembly: the units of an instance partition its page tokens
    (nothing lost, nothing twice), in nearly equal shares, whatever the chunk lengths."""
    cfg = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, 1, 10, 192)
    toks, items = mk.plan_decode_units(cfg, [1000] * 10, batch=1, q_len=64)
    assert sum(toks) == 10000 and len(toks) == 32                  # 8 KV heads x 32 units = 256 workgroups
    body = toks[:-1]                                               # the last unit also streams the tail
    assert max(body) - min(body) <= 8 and toks[-1] <= max(body)
    assert all(1 <= i <= 2 for i in items[:-1])                    # a unit spans at most two 1000-token pages
    # ragged chunk lengths, including a 1-token chunk; forced unit counts
    for units in (1, 3, 7, 64):
        cfg = mk.make_config(2, 8, 2, 128, 512, "bf16", 500000.0, 4, 6, 64, decode_units=units)
        lens = [300, 77, 1, 129, 1000, 5]
        toks, items = mk.plan_decode_units(cfg, lens, batch=3, q_len=9)
        assert sum(toks) == sum(lens) and 1 <= len(toks) <= units
        assert all(t >= 0 for t in toks) and all(i >= 0 for i in items)
    # batch 16: one unit per (instance, KV head) pair is already 128 workgroups -> 2 units each
    cfg = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, 16, 5, 192)
    toks, _ = mk.plan_decode_units(cfg, [1000] * 5, batch=16, q_len=100)
    assert len(toks) == 2 and sum(toks) == 5000
    # no pages at all: a single unit that only owns the tail
    toks, items = mk.plan_decode_units(cfg, [], batch=1, q_len=10)
    assert toks == [0] and items == [0]
    with pytest.raises(mk.MatKVError):
        mk.plan_decode_units(cfg, [0, 5], batch=1, q_len=10)


def test_decode_partition_over_compressed_pages(mk):
    """Host logic: over compressed pages the unit with the tail has up to 128 page tokens fewer than over plain ones, the others share them
    evenly, and there are as many units, also where the configuration fixes a number of them that leaves each a few tokens.  Units of
    several pages have to have 192 tokens for that, of one page 128."""
    rng = np.random.default_rng(5)
    spared = short = 0
    for trial in range(400):
        units = int(rng.choice([0, 0, 1, 2, 3, 7, 16, 64]))
        max_tail = int(rng.choice([8, 24, 128, 512]))
        lens = [int(n) for n in rng.integers(1, int(rng.choice([30, 300, 2000])) + 1, size=int(rng.integers(0, 7)))]
        batch, q = int(rng.integers(1, 5)), int(rng.integers(1, max_tail + 1))
        cfg = mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, 4, 6, max_tail, decode_units=units)
        plain, _ = mk.plan_decode_units(cfg, lens, batch, q)
        codes, _ = mk.plan_decode_units(cfg, lens, batch, q, mk.PAGE_E4M3)
        assert len(codes) == len(plain) and sum(codes) == sum(plain) == sum(lens)
        tail = q + (max_tail - q) // 2
        if len(plain) == 1 or tail * len(plain) >= sum(lens) + tail or sum(lens) + tail < (192 if len(lens) > 1 else 128) * len(plain):
            assert codes == plain
            short += len(plain) > 1
        else:
            ragged = 8 + 7 * len(lens)                     # (granules of eight tokens, a page's last one may hold one)
            assert -ragged <= plain[-1] - codes[-1] <= 128 + ragged and codes[-1] <= codes[0] + ragged
            assert max(codes[:-2] + codes[:1]) - min(codes[:-2] + codes[:1]) <= ragged
            spared += 1
    assert spared > 50 and short > 30
    cfg = mk.make_config(2, 16, 4, 128, 4096, "bf16", 500000.0, 1, 1, 8, decode_units=16)
    assert len(mk.plan_decode_units(cfg, [200], 1, 4, mk.PAGE_E4M3)[0]) == 16
    for lens, spares in (([214] * 3, False), ([642], True), ([88] * 8, False), ([1295] * 4, False), ([1295] * 5, True)):
        cfg = mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, 1, 8, 72)
        assert (mk.plan_decode_units(cfg, lens, 1, 64, mk.PAGE_E4M3) != mk.plan_decode_units(cfg, lens, 1, 64)) == spares
    with pytest.raises(mk.MatKVError):
        mk.plan_decode_units(cfg, [200], 1, 4, 2)
    with pytest.raises(mk.MatKVError):
        mk.plan_decode_units(mk.make_config(2, 4, 2, 64, 256, "f32", 10000.0, 1, 1, 8), [200], 1, 4, mk.PAGE_E4M3)


def test_decode_partition_never_exceeds_the_compute_units(mk):
    """Workgroups of a decode launch = units x KV heads over the batch: at most 256, so that no
    compute unit holds two (batch 3 x 8 KV heads: 10 units each, not 11)."""
    for batch in (1, 2, 3, 5, 7, 16):
        cfg = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, batch, 10, 192)
        toks, _ = mk.plan_decode_units(cfg, [1000] * 10, batch=batch, q_len=64)
        assert len(toks) * batch * 8 <= 256 and len(toks) == 256 // (batch * 8)
        assert sum(toks) == 10000


def test_even_partition_covers_every_instance_once(mk):
    """Host logic of the even decode partition: runs in number always 256 / KV heads; every page token of an instance streamed by exactly
    one run that lists it; one tail per run and two users at most; an instance's tail in exactly one of its runs; its partial slots used
    up by its runs' entries, the slots of all instances one behind the other; no run longer than the cut and a tail.  Instances without
    pages, single tokens and tails longer than a run among them."""
    rng = np.random.default_rng(11)
    built = chosen = 0
    for G, Hkv in ((4, 8), (8, 8), (3, 8), (8, 2), (1, 16)):
        for trial in range(24):
            batch = int(rng.integers(2, min(256 // Hkv, 40) + 1))
            most = int(rng.choice([3, 200, 4000]))
            pages = [[int(rng.integers(1, most + 1)) for _ in range(int(rng.integers(0, 5)))] for _ in range(batch)]
            max_tail = int(rng.choice([16, 128, 2048]))
            q_lens = [int(rng.integers(1, max_tail + 1)) for _ in range(batch)]
            cfg = mk.make_config(2, G * Hkv, Hkv, 128, 4096, "bf16", 500000.0, batch, 4, max_tail)
            runs, slots, taken = mk.plan_even_units(cfg, pages, q_lens)
            if batch <= 4 and G <= 4:
                assert runs == [] and not taken             # (one launch per step)
                continue
            built += 1
            chosen += taken
            assert len(runs) == 256 // Hkv
            seen, used, tails = [0] * batch, [set() for _ in range(batch)], [0] * batch
            tail_tokens = [(q + (max_tail - q) // 2 + 7) // 8 * 8 for q in q_lens]
            total = sum(sum((n + 7) // 8 * 8 for n in p) for p in pages) + sum(tail_tokens)
            for r in runs:
                assert len(r["users"]) <= 2 and r["tokens"] == sum(n for _, _, n in r["users"])
                assert len({b for b, _, _ in r["users"]}) == len(r["users"])
                if r["tail"] is not None:
                    assert r["tail"] in [b for b, _, _ in r["users"]]
                    tails[r["tail"]] += 1
                for b, slot, n in r["users"]:
                    assert n > 0 or r["tail"] == b
                    seen[b] += n
                    assert slot not in used[b] and slots[b][0] <= slot < slots[b][0] + slots[b][1]
                    used[b].add(slot)
            assert seen == [sum(p) for p in pages] and tails == [1] * batch
            assert [len(u) for u in used] == [c for _, c in slots]
            assert [f for f, _ in slots] == [sum(c for _, c in slots[:b]) for b in range(batch)]
            empty = [not r["users"] for r in runs]
            assert empty == sorted(empty)                   # empty runs come last
            assert max(r["tokens"] for r in runs) <= 8 * max(16, -(-total // 8 // len(runs)) * 2 + max(tail_tokens) // 8)
    assert built > 100 and 10 < chosen < built
    cfg = mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, 6, 2, 64, decode_units=3)
    assert mk.plan_even_units(cfg, [[500]] * 6, [9] * 6) == ([], None, False)
    for bad in (([[0]] * 6, [9] * 6), ([[5]] * 6, [65] * 6), ([[5]] * 7, [9] * 7)):
        with pytest.raises(mk.MatKVError):
            mk.plan_even_units(mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, 6, 2, 64), *bad)


def test_even_partition_is_taken_where_its_longest_run_is_shorter(mk):
    """Host logic: the choice between the two decode partitions.  Long tails, which are not cut, make runs as long as the units they
    replace: then the units stay."""
    def taken(caches, q_len, max_tail, Hq=32, fmt=mk.PAGE_PLAIN):
        cfg = mk.make_config(2, Hq, 8, 128, 4096, "bf16", 500000.0, len(caches), 3, max_tail)
        return mk.plan_even_units(cfg, caches, [q_len] * len(caches), fmt)[2]

    for Hq in (32, 64):
        assert taken([[3600]] * 17, 64, 256, Hq) and taken([[3600]] * 12, 64, 256, Hq) and taken([[900] * 3] * 20, 64, 256, Hq)
        assert taken([[1080 + 90 * b] for b in range(17)], 64, 256, Hq)
        assert not taken([[3600]] * 9, 64, 256, Hq) and not taken([[3600]] * 5, 64, 256, Hq) and not taken([[400]] * 24, 64, 256, Hq)
        assert not taken([[3600]] * 16, 64, 256, Hq) and not taken([[3600]] * 32, 64, 256, Hq)
        # longest run / longest unit: 2224 / 2224, 1120 / 1120, 1230 / 1230 tokens
        assert not taken([[200]] * 17, 2000, 2048, Hq) and not taken([[500]] * 20, 600, 640, Hq) and not taken([[300]] * 18, 900, 960, Hq)
        assert not taken([[510]] * 7, 1488, 1552, Hq) and not taken([[3577]] * 5, 982, 992, Hq)
        # 448 tokens fewer
        assert taken([[850]] * 17, 64, 256, Hq) and not taken([[850]] * 17, 64, 256, Hq, mk.PAGE_E4M3) and taken([[1200]] * 17, 64, 256, Hq, mk.PAGE_E4M3)


def test_decode_streams_only_rows_that_displace_something(mk):
    """Host logic: the cache's rows pass the last-level cache (256 MB) by where a step over all layers does not fit there and the weights do,
    or where the rows of one layer are many, and only while most of the chip walks to the end; short contexts of a whole model,
    whose weights alone exceed it, and launches of few workgroups or with one long walk take the ordinary loads."""
    shapes = {"3b": (28, 24, 3072), "8b": (32, 32, 4096), "70b": (80, 64, 8192)}

    def streams(model, tokens, batch=1, layers=None, fmt=mk.PAGE_PLAIN, question=32, units=0):
        n, Hq, hidden = shapes[model]
        cfg = mk.make_config(layers or n, Hq, 8, 128, hidden, "bf16", 500000.0, batch, 8, (question + 39) // 8 * 8, decode_units=units)
        return mk.plan_decode_streams(cfg, [[(b, tokens)] for b in range(batch)], [question] * batch, fmt)

    for model in shapes:
        for batch, tokens in ((1, 1), (1, 300), (3, 1000), (1, 4000), (16, 300)):
            assert not streams(model, tokens, batch)
        for batch, tokens in ((1, 1), (1, 3000), (3, 1000), (8, 100)):
            assert not streams(model, tokens, batch, fmt=mk.PAGE_E4M3)
        for batch, tokens in ((1, 8000), (8, 1500), (16, 5000), (17, 4000)):
            assert streams(model, tokens, batch) and streams(model, tokens // 2, batch, fmt=mk.PAGE_E4M3)
        # 136, 160, 192 and 232 workgroups
        assert not streams(model, 4000, 17, units=1) and not streams(model, 4000, 20, units=1) and not streams(model, 4000, 24, units=1)
        assert streams(model, 4000, 29, units=1) and not streams(model, 4000, 17, layers=4, units=1)
        assert streams(model, 4000, 20, layers=4, units=1) and streams(model, 4000, 24, layers=4, units=1)
        # one workgroup of each user walks the whole question
        assert streams(model, 4000, 8, layers=4) and not streams(model, 500, 8, question=2000) and not streams(model, 2000, 8, layers=4, question=2000)
    # slices of a model: all of it fits, the weights fit (16 layers of 8B: exactly), they nearly do
    assert not streams("8b", 4000, layers=8) and streams("8b", 5000, layers=8) and streams("8b", 3500, layers=16)
    assert not streams("8b", 100, layers=16) and not streams("8b", 2000, layers=17) and streams("8b", 4000, layers=17)
    # a batch that shares its pages streams them once
    cfg = mk.make_config(4, 32, 8, 128, 4096, "bf16", 500000.0, 4, 8, 64)
    assert mk.plan_decode_streams(cfg, [[(b, 5000)] for b in range(4)], [32] * 4)
    assert not mk.plan_decode_streams(cfg, [[(0, 5000)]] * 4, [32] * 4)
    # pages with more users than a tile has rows are walked by several units, which find them in the cache: four users of a page are one unit's
    # at four heads per KV head, and two units' at eight
    for model, Hq in (("8b", 32), ("70b", 64)):
        cfg = mk.make_config(4, Hq, 8, 128, 4096, "bf16", 500000.0, 16, 16, 64)
        for fmt, n in ((mk.PAGE_PLAIN, 1500), (mk.PAGE_E4M3, 3000)):
            quads = [[(16 * (b // 4) + i, n) for i in range(12)] for b in range(16)]
            assert mk.plan_decode_streams(cfg, quads, [32] * 16, fmt) == (Hq == 32)
            assert mk.plan_decode_streams(cfg, [[(16 * b + i, n) for i in range(3)] for b in range(16)], [32] * 16, fmt)
    cfg = mk.make_config(4, 32, 8, 128, 4096, "bf16", 500000.0, 4, 8, 64)
    for bad in (([[(0, 0)]], [4]), ([[(-1, 5)]], [4]), ([[(0, 5)]], [0]), ([[(0, 5)]], [65]), ([[(0, 5)]], [4], 7)):
        with pytest.raises(mk.MatKVError):
            mk.plan_decode_streams(cfg, *bad)


def test_fused_step_over_shared_pages_decides_for_its_own_walk(mk):
    """Host logic: a fused decode step beside a shared partition walks a shared page once for each of its users.  Where that is more than 9/8 of the
    distinct tokens and the weights alone exceed the last-level cache its rows stay there, whatever launches over the shared units
    do; where it is fewer, where the weights fit (8 and 16 layers), and where the step is not that launch, both say the same."""
    def plans(common, own, batch=2, layers=32, Hq=32, fmt=mk.PAGE_PLAIN):
        cfg = mk.make_config(layers, Hq, 8, 128, {24: 3072, 32: 4096, 64: 8192}[Hq], "bf16", 500000.0, batch, 2, 64)
        ids = [[(0, common), (1 + b, own)] for b in range(batch)]
        assert mk.plan_shared_units(cfg, ids, [32] * batch)[0]
        return mk.plan_decode_streams(cfg, ids, [32] * batch, fmt), mk.plan_step_streams(cfg, ids, [32] * batch, fmt)

    for layers in (18, 32):
        for own in (2500, 4000):                                    # 1.4 to 1.5 tokens walked per distinct one
            assert plans(5000, own, layers=layers) == (True, False)
        assert plans(3500, 3000, 4, layers) == (True, False) and plans(9000, 4000, layers=layers, fmt=mk.PAGE_E4M3) == (True, False)
        assert plans(700, 6000, layers=layers) == (True, True)      # 1.06
        assert plans(700, 6000, 6, layers) == (True, True)          # two launches: five users and more, eight heads to a KV head, many shared pages
        assert plans(5000, 4000, layers=layers, Hq=64) == (True, True) and plans(6000, 4000, layers=layers) == (True, True)
    for layers in (8, 16):
        assert plans(5000, 4000, layers=layers) == (True, True) and plans(3500, 3000, 4, layers) == (True, True)
    assert plans(5000, 4000, layers=2) == (False, False)
    cfg = mk.make_config(4, 32, 8, 128, 4096, "bf16", 500000.0, 4, 8, 64)
    assert mk.plan_step_streams(cfg, [[(b, 5000)] for b in range(4)], [32] * 4)     # no shared pages
    with pytest.raises(mk.MatKVError):
        mk.plan_step_streams(cfg, [[(0, 5)]], [65])


def test_shared_partition_covers_every_instance_once(mk):
    """Host logic of the shared decode partition: built when the batch's distinct pages are at least
    a twentieth fewer tokens than all uses; every (instance, page token) is streamed by exactly one
    unit that lists the instance; a unit has at most 16 / G users and at most one tail; every
    instance's tail sits in exactly one unit; every instance owns a run of distinct partial slots
    that its units' entries use up exactly; the launch has at most one workgroup per compute unit."""
    rng = np.random.default_rng(7)
    for G, Hkv in ((4, 8), (1, 2), (3, 8), (8, 8), (2, 4)):
        for trial in range(8):
            batch = int(rng.integers(2, 17))
            n_chunks = int(rng.integers(1, 7))
            lens = [int(rng.integers(1, 1500)) for _ in range(n_chunks)]
            pages = []
            for _ in range(batch):
                k = int(rng.integers(0, n_chunks + 1))
                ids = sorted(rng.choice(n_chunks, size=k, replace=False).tolist())
                if 0 not in ids and rng.random() < 0.8:
                    ids = [0] + ids                         # a hot chunk
                pages.append([(i, lens[i]) for i in ids])
            q_lens = [int(rng.integers(1, 100)) for _ in range(batch)]
            cfg = mk.make_config(2, G * Hkv, Hkv, 128, 4096, "bf16", 500000.0, batch, 6, 128)
            units, slots = mk.plan_shared_units(cfg, pages, q_lens)
            all_tokens = sum(n for p in pages for _, n in p)
            distinct = sum(lens[i] for i in {i for p in pages for i, _ in p})
            if 20 * distinct > 19 * all_tokens:
                assert units == [] and slots is None
                continue
            assert units and len(units) * Hkv <= 256
            streamed = [0] * batch
            used = [set() for _ in range(batch)]
            tails = [0] * batch
            for u in units:
                assert 1 <= len(u["users"]) <= 16 // G
                assert u["tokens"] > 0 or u["tail"] is not None
                if u["tail"] is not None:
                    assert u["tail"] in [inst for inst, _, _ in u["users"]]
                    tails[u["tail"]] += 1
                assert len({inst for inst, _, _ in u["users"]}) == len(u["users"])
                for inst, slot, seen in u["users"]:
                    assert 0 <= seen <= u["tokens"]
                    streamed[inst] += seen
                    first, count = slots[inst]
                    assert first <= slot < first + count and slot not in used[inst]
                    used[inst].add(slot)
            assert tails == [1] * batch
            assert streamed == [sum(n for _, n in p) for p in pages]
            assert [len(s) for s in used] == [c for _, c in slots]
            ends = sorted((f, f + c) for f, c in slots)
            assert all(a[1] == b[0] for a, b in zip(ends, ends[1:])) and ends[0][0] == 0     # the runs tile 0 .. total
            # every distinct page is streamed once per group of 16 / G users
            groups = sum(-(-sum(1 for p in pages if any(i == c for i, _ in p)) // (16 // G)) * lens[c]
                         for c in {i for p in pages for i, _ in p})
            assert sum(u["tokens"] for u in units) == groups
    # BASELINE config 3 (batch 16, five chunks each out of 200: 65 distinct of 80): 32 even units per KV head
    from workload import CONFIGS, question_lengths, retrieved_chunks
    s3 = CONFIGS[3]
    cfg = mk.make_config(32, 32, 8, 128, 4096, "bf16", 500000.0, 16, 5, 192)
    units, slots = mk.plan_shared_units(cfg, [[(c, 1000) for c in r] for r in retrieved_chunks(s3)], question_lengths(s3))
    assert len(units) == 32 and sum(u["tokens"] for u in units) == 65000
    sizes = [u["tokens"] for u in units]
    assert max(sizes) - min(sizes) <= 2 * 192               # a unit holds at most one tail (uncut, at most 192 rows) and ends before a second
    # not built: explicit unit count, fp32, a batch of one
    pages = [[(0, 500)], [(0, 500)], [(0, 500)]]
    assert mk.plan_shared_units(mk.make_config(2, 8, 2, 128, 512, "bf16", 500000.0, 3, 2, 64, decode_units=2), pages, [3, 3, 3])[0] == []
    assert mk.plan_shared_units(mk.make_config(2, 8, 2, 64, 512, "f32", 10000.0, 3, 2, 64), pages, [3, 3, 3])[0] == []
    assert mk.plan_shared_units(mk.make_config(2, 8, 2, 128, 512, "bf16", 500000.0, 3, 2, 64), pages[:1], [3])[0] == []
    units, _ = mk.plan_shared_units(mk.make_config(2, 8, 2, 128, 512, "bf16", 500000.0, 3, 2, 64), pages, [3, 3, 3])
    assert units and sum(u["tokens"] for u in units) == 500 and all(len(u["users"]) <= 4 for u in units)
    with pytest.raises(mk.MatKVError):
        mk.plan_shared_units(mk.make_config(2, 8, 2, 128, 512, "bf16", 500000.0, 3, 2, 64), [[(0, 0)], [(0, 5)]], [3, 3])


def test_prefill_layout_takes_short_tiles_for_short_questions(mk):
    """Host logic of the question prefill's layout: 64-row tiles only for questions of at most 64 (question row,
    query head) rows in units of at most 64 pieces, and there where the launch is a few short walks or two workgroups
    a compute unit shorten them."""
    def plan(batch, lens, q, Hq=32, fmt=mk.PAGE_PLAIN, dtype="bf16", D=128):
        cfg = mk.make_config(2, Hq, 8, D, 4096, dtype, 500000.0, batch, max(len(lens), 1), 224)
        return mk.plan_prefill(cfg, [lens] * batch, [q] * batch, fmt)

    for Hq, q in ((32, 1), (32, 16), (64, 1), (64, 8), (24, 1), (24, 21), (8, 64)):
        rows, units = plan(1, [64], q, Hq)
        assert (rows, units) == (64, [1]), (Hq, q)
        rows, units = plan(4, [1000] * 3, q, Hq)
        assert (rows, units) == (64, [8] * 4), (Hq, q)
        rows, units = plan(1, [1000] * 10, q, Hq)
        assert (rows, units) == (64, [32]), (Hq, q)
    assert plan(4, [1000] * 3, 17)[0] == 128 and plan(4, [1000] * 3, 16)[0] == 64      # 68 and 64 rows
    assert plan(4, [1000] * 3, 9, 64)[0] == 128 and plan(4, [1000] * 3, 22, 24)[0] == 128
    # many long walks of compressed pages: one unit each would leave compute units idle, two are one round of 64-row tiles
    assert plan(23, [735] * 6, 4, 32, mk.PAGE_E4M3) == (64, [2] * 23)
    assert plan(16, [270] * 15, 8, 64, mk.PAGE_E4M3) == (64, [4] * 16)
    assert plan(1, [1000], 64, 32, mk.PAGE_E4M3)[0] > 64 and plan(4, [1000] * 3, 17, 32, mk.PAGE_E4M3)[0] > 64
    assert plan(1, [], 5) == (64, [1])                          # no pages: the question alone
    assert plan(1, [1] * 300, 1)[0] == 0                        # units of more than 64 pieces
    assert plan(1, [100], 4, dtype="f32", D=64)[0] == 0         # row-per-workgroup kernel
    # one long question among short ones
    cfg = mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, 3, 3, 224)
    assert mk.plan_prefill(cfg, [[1000] * 3] * 3, [1, 40, 3])[0] == 128
    for bad in (([[1000]], [0]), ([[0]], [4]), ([[1000]], [225])):
        with pytest.raises(mk.MatKVError):
            mk.plan_prefill(cfg, *bad)


def test_prefill_layout_estimate_costs_little(mk):
    """Host time: the estimate of the launch's time (from 640 tokens on) adds less than half of what a layout takes without it (with every
    candidate dealt out it doubled it).  Best of many calls, the two lengths in turn."""
    import ctypes
    import time
    i32, B, n = ctypes.c_int32, 4, 3
    cfg = mk.make_config(2, 32, 8, 128, 4096, "bf16", 500000.0, B, n, 256)

    def call(tokens):
        lens = [(tokens - 70) // n] * (n - 1)
        args = (i32 * (B * n))(*((lens + [tokens - 70 - sum(lens)]) * B)), (i32 * B)(*[n] * B), (i32 * B)(*[70] * B), B, 0, None
        t0 = time.perf_counter()
        for _ in range(50):
            assert mk.lib().matkv_plan_prefill(ctypes.byref(cfg), *args) > 0
        return time.perf_counter() - t0

    for attempt in range(3):                                # (another process may be at work)
        times = [(call(639), call(640)) for _ in range(100)]
        without, with_estimate = (min(t) for t in zip(*times))
        if with_estimate < 1.5 * without:
            return
    raise AssertionError(f"{with_estimate / without:.2f} times")


def test_prefill_layout_does_not_cut_short_caches_of_a_large_batch(mk):
    """Host logic: a batch whose row tiles alone nearly fill the chip is cut only into units of 256 tokens and
    more (a cut of a short cache costs more in partials than it saves); smaller batches into units of 128."""
    def units(batch, lens, q, Hq=32):
        cfg = mk.make_config(2, Hq, 8, 128, 4096, "bf16", 500000.0, batch, len(lens), 224)
        return mk.plan_prefill(cfg, [lens] * batch, [q] * batch)[1]

    for q in (1, 4, 16, 32):
        assert units(16, [150, 150], q) == [1] * 16
        assert units(12, [150, 150], q) == [1] * 12
        assert units(16, [250, 250 + 32 - q], q) == [2] * 16    # two units of 256 and more
        assert units(8, [150, 150], q) == [2 if q > 4 else 3] * 8       # (64-row tiles, two a compute unit: down to 96)
    assert units(1, [150, 150], 32) == [2]
    assert units(16, [4] * 120, 20) == [2] * 16                 # a walk of many short pieces is long all the same
    assert units(16, [4] * 60, 16) == [2] * 16 and units(16, [16] * 30, 4) == [4] * 16
    assert units(16, [4] * 120, 16) == [1] * 16                 # (up to 64 rows another kernel takes it, uncut)


def test_prefill_layout_over_many_pages(mk):
    """Host logic: units of more than 64 pieces stay on the row-tile kernels where those have workgroups enough
    and rows to fill them, and go to the other kernel otherwise."""
    def form(batch, n, tokens, q, Hq=32, fmt=mk.PAGE_PLAIN):
        cfg = mk.make_config(1, Hq, 8, 128, 4096, "bf16", 500000.0, batch, n, 224)
        return mk.plan_prefill(cfg, [[tokens] * n] * batch, [q] * batch, fmt)[0]

    for fmt in (mk.PAGE_PLAIN, mk.PAGE_E4M3):
        assert form(12, 150, 40, 64, 32, fmt) in (128, 256)     # 75 or 150 pieces a unit, enough workgroups
        assert form(3, 250, 64, 200, 24, fmt) in (128, 256)
        assert form(1, 300, 1, 64, 32, fmt) == 0                # a few workgroups
        assert form(24, 70, 8, 4, 32, fmt) == 0                 # tiles of mostly padding
        assert form(24, 60, 8, 4, 32, fmt) != 0                 # up to 64 pieces: always tiles


def test_projection_forms(mk):
    """Host logic: the split-axis form while its workgroups (eight per KV head and 32 rows) have a compute unit
    each, tiles beyond; small row counts and other shapes on the forms for them."""
    ROWS, GEMV, FEW, STAGED, TILES = range(5)

    def form(rows, Hkv=8, hidden=4096, dtype="bf16", D=128):
        return mk.plan_projection(mk.make_config(1, Hkv, Hkv, D, hidden, dtype, 10000.0, 1, 1, 64), rows)

    for hidden in (1024, 3072, 4096, 8192):
        for Hkv, last in ((1, 512), (2, 512), (4, 256), (6, 160), (8, 128), (16, 128)):
            assert form(last, Hkv, hidden) == STAGED and form(17, Hkv, hidden) == STAGED
            assert form(last + 1, Hkv, hidden) == TILES
        assert form(4096, 8, hidden) == TILES and form(16, 8, hidden) == FEW
    assert form(1) == GEMV and form(7) == GEMV and form(8) == FEW and form(1, hidden=8192) == FEW
    assert form(15, hidden=4608) == ROWS and form(16, hidden=4608) == TILES and form(3, hidden=6144) == GEMV
    assert form(100, dtype="f32", D=64, hidden=256) == ROWS and form(100, D=64, hidden=4096) == GEMV and form(100, D=64, hidden=512) == ROWS
    with pytest.raises(mk.MatKVError):
        form(0)


def test_projection_waits_for_its_draw_behind_the_last_products(tmp_path):
    """Device code of the split projection tiles: between a wave's draw and its last matrix instruction the compiler puts no wait for loads of its own
    (the kernel's are written out), so the last steps are multiplied as they arrive.  The others arrive behind their last product."""
    import subprocess
    from paper_2512_22195_amd.build import CSRC, FLAGS, hipcc
    asm = str(tmp_path / "tiles.s")
    subprocess.run([hipcc()] + FLAGS + ["--cuda-device-only", "-S", os.path.join(CSRC, "materialize_mfma.hip"), "-o", asm],
                   check=True, capture_output=True)
    with open(asm) as f:
        kernels = re.findall(r"^\S*materialize_tile_kernelILi(\d)ELi\dELi2ELb([01])E\S*:.*?\n(.*?)\.Lfunc_end", f.read(), re.S | re.M)
    assert sorted((int(mi), int(drawn)) for mi, drawn, _ in kernels) == [(1, 0), (2, 0), (3, 0), (4, 0), (4, 1), (5, 1), (6, 1), (8, 1)]
    for mi, drawn, body in kernels:
        lines = re.sub(r";;#ASMSTART.*?;;#ASMEND", "", body, flags=re.S).splitlines()
        draw = next(i for i, l in enumerate(lines) if "global_atomic_add" in l and "sc0" in l)
        products = [i for i in range(draw, len(lines)) if "v_mfma" in lines[i]]
        assert bool(products) == (drawn == "1")
        assert not [l for l in lines[draw:max(products, default=draw)] if "vmcnt" in l], mi
