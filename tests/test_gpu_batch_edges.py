"""Batched lookups at the edges of their tiles: counts around a tile's keys,
filters without keys, more tiles than the persistent grid has turns in
flight, keys and results at odd addresses; and lookups in filters that fit the
LDS, and adds into them, at the edges of their sizes; bit-exact against the CPU oracle.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import log, to_device
from oracle import parallel as oracle_par
from paper_2512_15595_amd import workloads

pytestmark = pytest.mark.gpu

KIB = 1 << 10
# (filter bytes, keys): the first filter has no keys (the padding slots name it)
FILTERS = [(64, 0), (32, 1), (4 * KIB, 255), (96, 256), (300 * KIB, 257), (8 * KIB, 511), (64 * KIB, 512),
           (5 << 20, 513), (16 * KIB, 0), (1 << 20, 1023), (160, 1024), (64 * KIB + 128, 1025),
           (2 << 20, 20_011), (48 * KIB, 100_003), (80 * KIB, 32_768), (80 * KIB + 256, 32_769), (96 * KIB, 4_000),
           (128 * KIB, 65_537), (160 * KIB, 2_049), (160 * KIB + 256, 6_000), (164, 5_000)]
MANY = [(256 * KIB, 700_001), (32 * KIB, 1_300_003), (2 << 20, 2_200_005)]  # 8,205 tiles of 512 keys


@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (8, 32, 9), (1, 32, 4), (4, 64, 16), (16, 64, 16)])
@pytest.mark.parametrize("many", [False, True])
def test_batched_lookup_at_tile_edges(s, S, k, many):
    from paper_2512_15595_amd import bf

    shapes = FILTERS + (MANY if many else [])
    block = s * S // 8
    blocks = [max(1, nbytes // block) for nbytes, _ in shapes]
    counts = [n for _, n in shapes]
    offsets = np.concatenate([[0], np.cumsum(counts)])
    total = int(offsets[-1])
    log(f"batched lookup edges s={s} S={S} k={k}: {len(shapes)} filters, {total} keys")
    g = workloads.rng(s + S + k)
    keys = g.integers(0, 2**64, size=total, dtype=np.uint64)
    # three quarters of the bits set: both results occur
    words = [g.integers(0, 256, size=nb * block, dtype=np.uint8) | g.integers(0, 256, size=nb * block, dtype=np.uint8)
             for nb in blocks]
    want = np.concatenate([oracle_par.contains(words[i], nb, s, S, k, i, keys[offsets[i]:offsets[i + 1]])
                           for i, nb in enumerate(blocks) if counts[i] > 0])
    filters = [bf.BloomFilter(nb, s, S, k, i) for i, nb in enumerate(blocks)]
    try:
        for f, w in zip(filters, words):
            f.load_words(torch.from_numpy(w).to("cuda"))
        d = to_device(keys, offset_elems=1)
        out = torch.full((total + 32,), 7, dtype=torch.uint8, device="cuda")
        plan = bf.BatchPlan(bf.BF_OP_CONTAINS, filters, d, offsets, out[3:total + 3])
        try:
            for launch in (plan.launch, plan.launch_direct):
                out.fill_(7)
                launch()
                got = out.cpu().numpy()
                assert np.array_equal(got[3:total + 3], want)
                assert (got[:3] == 7).all() and (got[total + 3:] == 7).all()
        finally:
            plan.close()
    finally:
        for f in filters:
            f.close()


@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (8, 32, 9), (1, 32, 4), (4, 64, 16)])
@pytest.mark.parametrize("nbytes,n", [(68, (1 << 22) + 1), (16 * KIB, (1 << 22) + 4_095), (17 * KIB + 36, 1 << 21),
                                      (80 * KIB, (1 << 21) + 2_049), (80 * KIB + 64, 1 << 22),
                                      (160 * KIB, 17_000_001), (160 * KIB + 64, 1 << 21)])
def test_lookup_in_lds_equals_the_oracle(s, S, k, nbytes, n):
    """The direct lookup's bytes too (a mapping of the caller's takes it)."""
    from paper_2512_15595_amd import bf

    block = s * S // 8
    nb = max(1, nbytes // block)
    log(f"lookup in LDS s={s} S={S} k={k}: {nb * block} bytes, {n} keys")
    g = workloads.rng(nb + s)
    keys = g.integers(0, 2**64, size=n, dtype=np.uint64)
    words = g.integers(0, 256, size=nb * block, dtype=np.uint8) | g.integers(0, 256, size=nb * block, dtype=np.uint8)
    f = bf.BloomFilter(nb, s, S, k, nb)
    try:
        f.load_words(torch.from_numpy(words).to("cuda"))
        d = to_device(keys, offset_elems=1)
        out = torch.full((n + 32,), 7, dtype=torch.uint8, device="cuda")
        f.contains(d, out=out[3:n + 3])
        got = out.cpu().numpy()
        assert np.array_equal(got[3:n + 3], oracle_par.contains(words, nb, s, S, k, nb, keys))
        assert (got[:3] == 7).all() and (got[n + 3:] == 7).all()
        f.set_mapping(bf.BF_OP_CONTAINS, 1, s, 1)
        assert torch.equal(f.contains(d), out[3:n + 3])
    finally:
        f.close()


@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (8, 32, 9), (1, 32, 4), (2, 32, 4), (4, 64, 16)])
@pytest.mark.parametrize("nbytes,n", [(68, 5_000), (4 * KIB, 32_769), (17 * KIB + 36, 8 * 18 * KIB), (80 * KIB, 655_360),
                                      (80 * KIB + 64, 2_000_001), (160 * KIB, 1_310_720), (160 * KIB + 64, 1 << 21)])
def test_add_in_lds_equals_the_oracle(s, S, k, nbytes, n):
    """On a filter that holds bits already; half of the keys are one key."""
    from paper_2512_15595_amd import bf

    block = s * S // 8
    nb = max(1, nbytes // block)
    log(f"add in LDS s={s} S={S} k={k}: {nb * block} bytes, {n} keys")
    g = workloads.rng(nb + s)
    keys = g.integers(0, 2**64, size=n, dtype=np.uint64)
    keys[::2] = 77
    old = np.zeros(nb * block, dtype=np.uint8)
    old[::7] = 129
    f = bf.BloomFilter(nb, s, S, k, nb)
    try:
        f.load_words(torch.from_numpy(old).to("cuda"))
        f.add(to_device(keys, offset_elems=1))
        got = f.words().cpu().numpy().view(np.uint8)
        assert np.array_equal(got, oracle_par.filter_words(nb, s, S, k, nb, keys).view(np.uint8) | old)
    finally:
        f.close()


@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (8, 32, 9), (1, 32, 4), (4, 64, 16)])
def test_batched_add_in_lds_equals_the_oracle(s, S, k):
    """Small filters in LDS (one of them twice in the plan), larger ones by
    the partitioned construction or directly."""
    from paper_2512_15595_amd import bf

    shapes = [(4 * KIB, 200_001), (64 * KIB, 65_537), (0, 0), (80 * KIB, 700_000), (80 * KIB + 256, 10_000),
              (160 * KIB, 900_001), (160 * KIB + 256, 30_000), (68, 3), (1 << 20, 400_000), (4 * KIB, 5_000)]
    block = s * S // 8
    blocks = [max(1, nbytes // block) for nbytes, _ in shapes]
    offsets = np.concatenate([[0], np.cumsum([n for _, n in shapes])])
    keys = workloads.rng(s + S).integers(0, 2**64, size=int(offsets[-1]), dtype=np.uint64)
    log(f"batched add in LDS s={s} S={S} k={k}: {len(shapes)} filters, {keys.size} keys")
    filters = [bf.BloomFilter(nb, s, S, k, i) for i, nb in enumerate(blocks)]
    filters[-1].close()
    filters[-1] = filters[0]
    share = [keys[offsets[i]:offsets[i + 1]] for i in range(len(shapes))]
    share[0] = np.concatenate([share[0], share[-1]])
    try:
        d = to_device(keys, offset_elems=1)
        for mode in ("launch", "launch_direct"):
            for f in filters:
                f.clear()
            plan = bf.BatchPlan(bf.BF_OP_ADD, filters, d, offsets)
            try:
                getattr(plan, mode)()
                got = [f.words().cpu().numpy().view(np.uint8) for f in filters]
            finally:
                plan.close()
            for i, nb in enumerate(blocks[:-1]):
                want = (oracle_par.filter_words(nb, s, S, k, i, share[i]).view(np.uint8) if share[i].size
                        else np.zeros(nb * block, dtype=np.uint8))
                assert np.array_equal(got[i], want), f"filter {i}"
    finally:
        for f in filters[:-1]:
            f.close()


@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (8, 32, 9), (1, 32, 4), (4, 64, 16)])
def test_batched_lookup_in_lds_equals_the_oracle(s, S, k):
    """Enough keys in small filters that the plan tests them in LDS (the rule
    of bf_batch.hip: 2^23 keys over 96 filters of like counts)."""
    from paper_2512_15595_amd import bf

    block = s * S // 8
    sizes = [68, 4 * KIB, 17 * KIB + 36, 80 * KIB, 80 * KIB + 64, 160 * KIB, 160 * KIB + 64, 300 * KIB] * 12
    blocks = [max(1, nbytes // block) for nbytes in sizes]
    counts = [87_000 + 37 * i for i in range(len(sizes))]
    offsets = np.concatenate([[0], np.cumsum(counts)])
    total = int(offsets[-1])
    log(f"batched lookup in LDS s={s} S={S} k={k}: {len(sizes)} filters, {total} keys")
    g = workloads.rng(s + S + k)
    keys = g.integers(0, 2**64, size=total, dtype=np.uint64)
    words = [g.integers(0, 256, size=nb * block, dtype=np.uint8) | g.integers(0, 256, size=nb * block, dtype=np.uint8)
             for nb in blocks]
    want = np.concatenate([oracle_par.contains(words[i], nb, s, S, k, i, keys[offsets[i]:offsets[i + 1]])
                           for i, nb in enumerate(blocks)])
    filters = [bf.BloomFilter(nb, s, S, k, i) for i, nb in enumerate(blocks)]
    try:
        for f, w in zip(filters, words):
            f.load_words(torch.from_numpy(w).to("cuda"))
        out = torch.full((total + 32,), 7, dtype=torch.uint8, device="cuda")
        plan = bf.BatchPlan(bf.BF_OP_CONTAINS, filters, to_device(keys, offset_elems=1), offsets, out[3:total + 3])
        try:
            for launch in (plan.launch, plan.launch_direct):
                out.fill_(7)
                launch()
                got = out.cpu().numpy()
                assert np.array_equal(got[3:total + 3], want)
                assert (got[:3] == 7).all() and (got[total + 3:] == 7).all()
        finally:
            plan.close()
    finally:
        for f in filters:
            f.close()


@pytest.mark.parametrize("forced", [False, True])
@pytest.mark.parametrize("mode", ["launch", "launch_direct"])
def test_partitioned_plan_over_overlapping_words(mode, forced):
    """A dense filter named twice and two overlapping views of one buffer: no
    two workgroups of the construction may write back the same chunk."""
    from paper_2512_15595_amd import bf

    mib = 1 << 20
    words = torch.zeros(96 * mib, dtype=torch.uint8, device="cuda")
    # (first byte, bytes, keys); entry 2 is entry 0 again
    spec = [(0, 40 * mib, 1_500_001), (48 * mib, 48 * mib, 1_600_003), None, (64 * mib, 16 * mib, 300_007)]
    log(f"plan over overlapping words mode={mode} forced={forced}")
    filters = []
    for i, x in enumerate(spec):
        filters.append(filters[0] if x is None else
                       bf.BloomFilterView(words[x[0]:x[0] + x[1]], x[1] // 32, 8, 32, 8, i))
    spec[2] = (0, 40 * mib, 900_001)
    offsets = np.concatenate([[0], np.cumsum([n for _, _, n in spec])])
    keys = workloads.rng(17).integers(0, 2**64, size=int(offsets[-1]), dtype=np.uint64)
    want = np.zeros(96 * mib, dtype=np.uint8)
    for i, (at, nbytes, _) in enumerate(spec):
        want[at:at + nbytes] |= oracle_par.filter_words(nbytes // 32, 8, 32, 8, 0 if i == 2 else i,
                                                        keys[offsets[i]:offsets[i + 1]]).view(np.uint8)
    try:
        if forced:
            filters[0].set_mapping(bf.BF_OP_ADD, strategy=bf.BF_STRATEGY_PARTITIONED)
        plan = bf.BatchPlan(bf.BF_OP_ADD, filters, to_device(keys), offsets)
        try:
            info = plan.info()
            assert info.strategy == bf.BF_STRATEGY_PARTITIONED
            assert info.ntiles > 0, "the keys of entries that overlap an owner"
            getattr(plan, mode)()
            assert np.array_equal(words.cpu().numpy(), want)
        finally:
            plan.close()
    finally:
        for i in (0, 1, 3):
            filters[i].close()


@pytest.mark.parametrize("s,S,k,nbytes,per,count,lds", [
    (1, 32, 4, 128 * KIB, 8_192, 512, False), (4, 64, 16, 128 * KIB, 8_192, 512, False),
    (8, 32, 9, 64 * KIB, 2_100, 2000, False), (8, 32, 8, 32 * KIB, 8_192, 1024, True),
    (4, 64, 16, 32 * KIB, 8_192, 1024, True), (1, 64, 8, 32 * KIB, 8_192, 1024, True)])
def test_lookup_plans_take_lds_where_it_pays(s, S, k, nbytes, per, count, lds):
    """The rule follows the layout; the result does not depend on it.  Tiles
    hold 256 or 512 keys, items at least 4,096."""
    from paper_2512_15595_amd import bf

    block = s * S // 8
    total = per * count
    words = torch.randint(0, 256, (count * nbytes,), dtype=torch.uint8, device="cuda")
    filters = [bf.BloomFilterView(words[i * nbytes:(i + 1) * nbytes], nbytes // block, s, S, k, i) for i in range(count)]
    keys = torch.randint(-2**63, 2**63 - 1, (total,), dtype=torch.int64, device="cuda")
    out = torch.empty(total, dtype=torch.uint8, device="cuda")
    log(f"lookup plan rule s={s} S={S} k={k}: {count} filters of {nbytes} bytes, {per} keys each")
    try:
        plan = bf.BatchPlan(bf.BF_OP_CONTAINS, filters, keys, [i * per for i in range(count + 1)], out)
        try:
            tiles = sum(plan.info().tiles_per_class)
            assert (tiles < total // 2048) == lds, tiles
            plan.launch()
            for i in (0, 1, count // 2, count - 1):
                want = oracle_par.contains(words[i * nbytes:(i + 1) * nbytes].cpu().numpy(), nbytes // block, s, S, k, i,
                                           keys[i * per:(i + 1) * per].cpu().numpy().view(np.uint64))
                assert np.array_equal(out[i * per:(i + 1) * per].cpu().numpy(), want)
        finally:
            plan.close()
    finally:
        for f in filters:
            f.close()


def _plan_of(shapes, seed):
    """An add plan over filters (bytes, keys) of 32-byte blocks in one buffer."""
    from paper_2512_15595_amd import bf

    ends = np.concatenate([[0], np.cumsum([nbytes for nbytes, _ in shapes])])
    offsets = np.concatenate([[0], np.cumsum([n for _, n in shapes])])
    words = torch.zeros(int(ends[-1]), dtype=torch.uint8, device="cuda")
    filters = [bf.BloomFilterView(words[int(ends[i]):int(ends[i + 1])], nbytes // 32, 8, 32, 8, i)
               for i, (nbytes, _) in enumerate(shapes)]
    keys = workloads.rng(seed).integers(0, 2**64, size=int(offsets[-1]), dtype=np.uint64)
    d_keys = to_device(keys)
    free = torch.cuda.mem_get_info()[0]
    plan = bf.BatchPlan(bf.BF_OP_ADD, filters, d_keys, offsets)
    torch.cuda.synchronize()
    return plan, filters, words, ends, offsets, keys, free - torch.cuda.mem_get_info()[0]


def _check_plan(plan, filters, words, ends, offsets, keys, sample):
    plan.launch()
    for i in sample:
        want = oracle_par.filter_words((int(ends[i + 1]) - int(ends[i])) // 32, 8, 32, 8, i, keys[offsets[i]:offsets[i + 1]])
        assert np.array_equal(words[int(ends[i]):int(ends[i + 1])].cpu().numpy(), want.view(np.uint8)), f"filter {i}"


@pytest.mark.parametrize("count,nbytes,per", [(20_000, 4 * KIB, 110), (8_000, 32 * KIB, 600)])
def test_plans_of_many_filters_with_few_keys(count, nbytes, per):
    """A step of the construction holds one filter's keys and is stored whole:
    such plans go to tiles, which take a few bytes per key."""
    from paper_2512_15595_amd import bf

    log(f"add plan of {count} filters of {nbytes} bytes, {per} keys each")
    plan, *rest, taken = _plan_of([(nbytes, per)] * count, 5)
    try:
        assert plan.info().strategy == bf.BF_STRATEGY_DIRECT
        assert taken < 64 << 20
        _check_plan(plan, *rest, (0, 1, 77, count - 1))
    finally:
        plan.close()
        for f in rest[0]:
            f.close()


def test_plan_without_memory_for_the_construction_runs_in_tiles():
    """20,000 filters of 32 KiB and 2,000 keys want 1.6 GB; with less than that
    left the plan is made all the same."""
    from paper_2512_15595_amd import bf

    shapes = [(32 * KIB, 2_000)] * 20_000
    log("add plan with 1.6 GB of construction workspace and 1 GB of memory")
    plan, filters, words, ends, offsets, keys, _ = _plan_of(shapes, 6)
    assert plan.info().strategy == bf.BF_STRATEGY_PARTITIONED
    plan.close()
    d_keys = to_device(keys)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device="cuda")
    fillers = []  # what the library's pool still holds, but for 1 GB
    try:
        while True:
            try:
                fillers.append(bf.BloomFilter((256 << 20) // 32, 8, 32, 8, 0))
            except bf.BfError:
                break
        for f in fillers[-4:]:
            f.close()
        plan = bf.BatchPlan(bf.BF_OP_ADD, filters, d_keys, offsets)
        assert plan.info().strategy == bf.BF_STRATEGY_DIRECT
        _check_plan(plan, filters, words, ends, offsets, keys, (0, 19_999))
    finally:
        del hold
        torch.cuda.empty_cache()
        plan.close()
        for f in filters + fillers[:-4]:
            f.close()


@pytest.mark.parametrize("small,large,partitioned", [((64 * KIB, 8_192, 2048), (16 << 20, 1 << 22, 1), True),
                                                     ((128 * KIB, 16_384, 512), (4 << 20, 1 << 20, 4), True),
                                                     ((128 * KIB, 16_384, 512), (1 << 20, 1 << 20, 1), False)])
def test_small_filters_join_the_construction_where_it_pays(small, large, partitioned):
    """Beside many small filters that fit the LDS, a few large ones are too
    little for a construction of their own and slow in tiles."""
    from paper_2512_15595_amd import bf

    shapes = [(small[0], small[1])] * small[2] + [(large[0], large[1])] * large[2]
    log(f"add plan of {small} and {large} (bytes, keys, filters)")
    plan, *rest, _ = _plan_of(shapes, 8)
    try:
        assert (plan.info().strategy == bf.BF_STRATEGY_PARTITIONED) == partitioned
        _check_plan(plan, *rest, (0, small[2] - 1, small[2], len(shapes) - 1))
    finally:
        plan.close()
        for f in rest[0]:
            f.close()


def test_joined_plan_without_memory_keeps_its_small_filters_in_lds():
    """2,048 filters of 64 KiB join the construction of one of 16 MiB; where
    its 0.4 GB are not to be had they run in LDS again, not in tiles."""
    from paper_2512_15595_amd import bf

    shapes = [(64 * KIB, 8_192)] * 2048 + [(16 << 20, 1 << 22)]
    log("add plan whose small filters would join the construction, and 0.1 GB of memory")
    plan, filters, words, ends, offsets, keys, _ = _plan_of(shapes, 9)
    assert plan.info().strategy == bf.BF_STRATEGY_PARTITIONED
    plan.close()
    d_keys = to_device(keys)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device="cuda")
    fillers = []
    try:
        while True:
            try:
                fillers.append(bf.BloomFilter((96 << 20) // 32, 8, 32, 8, 0))
            except bf.BfError:
                break
        fillers.pop().close()
        plan = bf.BatchPlan(bf.BF_OP_ADD, filters, d_keys, offsets)
        info = plan.info()
        assert info.strategy == bf.BF_STRATEGY_DIRECT
        # the tiles (256 or 512 keys) of the one filter that the LDS cannot hold
        assert sum(info.tiles_per_class) <= (1 << 22) // 256
        del hold
        _check_plan(plan, filters, words, ends, offsets, keys, (0, 2_047, 2_048))
    finally:
        hold = None
        torch.cuda.empty_cache()
        plan.close()
        for f in filters + fillers:
            f.close()


@pytest.mark.parametrize("nbytes,n", [(32 << 20, 1 << 26), (64 * KIB, 1 << 24)])
def test_per_filter_launches_take_the_route_of_single_calls(nbytes, n):
    """bf_batch_launch_per_filter is a bf_add / bf_contains per filter: grouped
    or in LDS where those are (2.4 and 1.6 times the direct kernels' rate), and
    with their results."""
    from paper_2512_15595_amd import bf

    keys = torch.randint(-2**63, 2**63 - 1, (n,), dtype=torch.int64, device="cuda")
    outs = [torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(2)]
    f, g = bf.BloomFilter(nbytes // 32, 8, 32, 8, 3), bf.BloomFilter(nbytes // 32, 8, 32, 8, 3)
    some = keys[:nbytes // 8].contiguous()
    add = bf.BatchPlan(bf.BF_OP_ADD, [f], some, [0, some.numel()])
    plan = bf.BatchPlan(bf.BF_OP_CONTAINS, [f], keys, [0, n], outs[0])
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best(call):
        times = []
        for _ in range(8):
            a.record()
            call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    try:
        add.launch_per_filter()
        g.add(some)
        assert torch.equal(f.words(), g.words())
        per_filter, single = best(plan.launch_per_filter), best(lambda: g.contains(keys, out=outs[1]))
        log(f"{n} lookups in {nbytes} bytes: per filter {per_filter:.3f} ms, bf_contains {single:.3f}")
        assert torch.equal(outs[0], outs[1])
        assert per_filter < 1.25 * single
    finally:
        add.close()
        plan.close()
        f.close()
        g.close()
