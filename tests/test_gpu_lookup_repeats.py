"""Grouped lookups of repeated keys: the sample that chooses between grouping
and direct lookups, keys beyond their run's clip, passes of one call, two
streams at once; bit-exact against the CPU oracle or the caller-mapped direct
lookup.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import log, to_device
from oracle import parallel as oracle_par
from paper_2512_15595_amd import workloads
from test_call_plan import CONTAINS, GROUPED, call_plan

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

MIB = 1 << 20
# filter bytes, keys: the least of every size that is grouped, one digit and two
SIZES = [(8 * MIB, 1 << 24), (16 * MIB + 96, (1 << 23) + 1), (33 * MIB, (3 << 21) + 77), (64 * MIB, (3 << 21) + 8191),
         (65 * MIB, 11_000_003)]


def _filter(nbytes, s=8, S=32, k=8, seed=5):
    """A filter with three quarters of the bits set, and its bytes."""
    from paper_2512_15595_amd import bf

    g = workloads.rng(nbytes % 1001 + s)
    block = s * S // 8
    nb = nbytes // block
    words = g.integers(0, 256, size=nb * block, dtype=np.uint8) | g.integers(0, 256, size=nb * block, dtype=np.uint8)
    f = bf.BloomFilter(nb, s, S, k, seed)
    f.load_words(torch.from_numpy(words).to("cuda"))
    return f, words, nb


def _repeated(n, share, distinct, seed):
    """n keys of which a share are copies of `distinct` ones."""
    g = workloads.rng(seed)
    keys = g.integers(0, 2**64, size=n, dtype=np.uint64)
    copies = g.random(n) < share
    keys[copies] = keys[:distinct][g.integers(0, distinct, size=int(copies.sum()))]
    return keys


@pytest.mark.parametrize("nbytes,n", SIZES)
@pytest.mark.parametrize("share,distinct", [(0.0, 1), (0.01, 1), (0.2, 3), (0.45, 2), (0.95, 100), (1.0, 1), (1.0, 5000)])
def test_lookups_of_repeated_keys(nbytes, n, share, distinct):
    assert call_plan(nbytes, CONTAINS, n).route == GROUPED
    assert call_plan(nbytes, CONTAINS, n // 2).route != GROUPED
    keys = _repeated(n, share, distinct, n)
    log(f"repeated lookups: {nbytes} bytes, {n} keys, {share} of them copies of {distinct}")
    f, words, nb = _filter(nbytes)
    try:
        out = torch.full((n + 32,), 7, dtype=torch.uint8, device="cuda")
        f.contains(to_device(keys, offset_elems=1), out=out[5:n + 5])
        got = out.cpu().numpy()
        assert np.array_equal(got[5:n + 5], oracle_par.contains(words, nb, 8, 32, 8, 5, keys))
        assert (got[:5] == 7).all() and (got[n + 5:] == 7).all()
    finally:
        f.close()


@pytest.mark.parametrize("s,S,k", [(1, 32, 4), (2, 64, 16), (8, 32, 9), (16, 64, 16), (16, 32, 17)])
@pytest.mark.parametrize("share", [0.02, 0.9])
@pytest.mark.parametrize("nbytes,n", [(33 * MIB, (3 << 21) + 5), (70 * MIB, 12_000_007)])
def test_repeated_lookups_of_other_layouts(s, S, k, share, nbytes, n):
    keys = _repeated(n, share, 7, s + k)
    log(f"repeated lookups s={s} S={S} k={k}: {nbytes} bytes, {n} keys, {share} copies")
    f, words, nb = _filter(nbytes, s, S, k)
    try:
        got = f.contains(to_device(keys)).cpu().numpy()
        assert np.array_equal(got, oracle_par.contains(words, nb, s, S, k, 5, keys))
    finally:
        f.close()


@pytest.mark.parametrize("nbytes,n,kind,most", [
    (32 * MIB, 1 << 26, "one", 2.0), (1024 * MIB, 1 << 26, "one", 2.0),
    # grouped they take 1.17 and 1.30 times as long as directly
    (32 * MIB, 1 << 26, "half", 1.12), (32 * MIB, 1 << 26, "skewed", 1.15)])
def test_repeated_keys_cost_what_direct_lookups_cost(nbytes, n, kind, most):
    """All keys equal: their line stays in the caches, and a direct lookup of
    them takes a quarter of the time that grouping does.  Half of them equal, or
    skewed: it is faster too."""
    from paper_2512_15595_amd import bf

    f, _, _ = _filter(nbytes)
    keys = torch.full((n,), 1234567, dtype=torch.int64, device="cuda")
    if kind == "half":
        keys[torch.rand(n, device="cuda") < 0.5] = 0
        keys += torch.randint(1, 2**62, (n,), device="cuda") * (keys == 0)
    elif kind == "skewed":
        keys = (torch.rand(n, device="cuda", dtype=torch.float64).pow(8) * 1e6).long()
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best():
        times = []
        for _ in range(8):
            a.record()
            f.contains(keys, out=out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    try:
        ms = best()
        f.set_mapping(bf.BF_OP_CONTAINS, 1, 8, 2)
        direct = best()
        log(f"{n} keys ({kind}) in {nbytes >> 20} MiB: {ms:.3f} ms, direct {direct:.3f}")
        assert ms < most * direct
    finally:
        f.close()


def test_lookup_of_more_keys_than_a_pass():
    """2^28 + 40,961 keys: the last pass would not be grouped by itself."""
    from paper_2512_15595_amd import bf

    n, nbytes = (1 << 28) + 40_961, 1536 * MIB  # 2^8 second digits
    assert call_plan(nbytes, CONTAINS, n).route == GROUPED
    log(f"lookup in two passes: {n} keys")
    f = bf.BloomFilter(nbytes // 32, 8, 32, 8, 3)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    keys = torch.randint(-2**63, 2**63 - 1, (n,), dtype=torch.int64, device="cuda", generator=g)
    try:
        f.add(keys[1::2].contiguous())
        got = f.contains(keys)
        assert bool(got[1::2].all())
        f.set_mapping(bf.BF_OP_CONTAINS, 1, 8, 2)
        assert torch.equal(f.contains(keys), got)
    finally:
        f.close()


def test_grouped_lookups_on_two_streams():
    """Two filters and one shared filter looked up from two streams at once:
    every call has a workspace of its own."""
    n, nbytes = (3 << 21) + 3, 40 * MIB
    fa, wa, nb = _filter(nbytes, seed=5)
    fb, wb, _ = _filter(nbytes, seed=5)
    keys = [_repeated(n, share, 4, 60 + i) for i, share in enumerate((0.0, 0.3, 0.9, 0.0))]
    dev = [to_device(k) for k in keys]
    want = {(f, i): oracle_par.contains(w, nb, 8, 32, 8, 5, keys[i]) for f, w in ((0, wa), (1, wb)) for i in range(4)}
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    log(f"grouped lookups on two streams: {n} keys each")
    torch.cuda.synchronize()
    outs = []
    try:
        for turn in range(3):
            for i in range(4):
                for f, filt in enumerate((fa, fb)):
                    st = streams[(f + i + turn) % 2]
                    out = torch.empty(n, dtype=torch.uint8, device="cuda")
                    st.wait_stream(torch.cuda.current_stream())
                    filt.contains(dev[i], out=out, stream=st)
                    outs.append((f, i, out))
        torch.cuda.synchronize()
        for f, i, out in outs:
            assert np.array_equal(out.cpu().numpy(), want[f, i]), (f, i)
    finally:
        fa.close()
        fb.close()


@pytest.mark.parametrize("nbytes", [64 * MIB + 64 * 1024, 66 * MIB, 130 * MIB])
def test_lookups_with_a_partial_last_high_digit(nbytes):
    """1 chunk of 64 in the last high digit, and halves: its runs are longer
    than those of the other digits and are clipped by a length of their own."""
    n = 13_000_003
    assert call_plan(nbytes, CONTAINS, n).route == GROUPED
    keys = _repeated(n, 0.0, 1, nbytes)
    log(f"partial last high digit: {nbytes} bytes, {n} keys")
    f, words, nb = _filter(nbytes)
    try:
        got = f.contains(to_device(keys)).cpu().numpy()
        assert np.array_equal(got, oracle_par.contains(words, nb, 8, 32, 8, 5, keys))
    finally:
        f.close()


def test_workspace_kept_by_lookups_is_given_back_to_filters():
    """The pool keeps a large lookup's workspace (5.8 GB) for the next one; a
    filter that needs the memory gets it."""
    from paper_2512_15595_amd import bf

    n = 1 << 28
    f = bf.BloomFilter((1 << 30) // 32, 8, 32, 8, 3)
    keys = torch.zeros(n, dtype=torch.int64, device="cuda")
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - (7 << 30), dtype=torch.uint8, device="cuda")
    made = []
    try:
        log("lookup with 7 GiB of memory left, then a filter of 5 GiB")
        f.contains(keys, out=out)
        torch.cuda.synchronize()
        made.append(bf.BloomFilter((5 << 30) // 32, 8, 32, 8, 4))
        f.contains(keys, out=out)  # no memory for a workspace now: directly
        assert not bool(out.any())
        made.pop().close()
        torch.cuda.synchronize()
        f.contains(keys, out=out)
        torch.cuda.synchronize()
        kept = torch.cuda.mem_get_info()[0]
        assert bf.bf_release_workspace() == bf.BF_OK
        assert torch.cuda.mem_get_info()[0] > kept + (4 << 30)
    finally:
        del hold
        torch.cuda.empty_cache()
        for x in made + [f]:
            x.close()
