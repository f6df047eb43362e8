"""Sorted-step grouping: the grouped lookup (bf_contains of many keys on a
filter beyond the L2) and the partitioned construction at the edges of their
steps (8,192 records), digits and runs, bit-exact against the CPU oracle.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import log, to_device
from oracle import parallel as oracle_par
from paper_2512_15595_amd import workloads

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

MIB = 1 << 20
STEP = 8192


def _bf():
    from paper_2512_15595_amd import bf

    return bf


def _dense_words(nbytes: int, seed: int) -> np.ndarray:
    """Filter bytes with three quarters of the bits set: every result occurs."""
    g = workloads.rng(seed)
    return g.integers(0, 256, size=nbytes, dtype=np.uint8) | g.integers(0, 256, size=nbytes, dtype=np.uint8)


def _keys(n: int, kind: str, seed: int) -> np.ndarray:
    g = workloads.rng(seed)
    if kind == "one":
        return np.full(n, 0x1234_5678_9ABC_DEF1, dtype=np.uint64)
    keys = g.integers(0, 2**64, size=n, dtype=np.uint64)
    if kind == "repeated":  # a fifth of the keys is one key, a tenth another
        r = g.random(n)
        keys[r < 0.2] = 77
        keys[r > 0.9] = 2**63
    return keys


# filter bytes, keys: the smallest taken, ragged ones, whole and partial last
# chunks, and the first filter that takes two digits
SIZES = [
    (16 * MIB, 1 << 22),
    (17 * MIB + 256, (1 << 22) + 1),
    (64 * MIB, (1 << 22) + STEP - 1),
    (64 * MIB + 256, (1 << 23) + (2 << 20)),
    (130 * MIB + 128 * 77, 13_000_001),
]


@pytest.mark.parametrize("nbytes,n", SIZES)
@pytest.mark.parametrize("s,S,k", [(8, 32, 8), (1, 32, 4), (2, 64, 16), (16, 64, 16), (4, 32, 5)])
def test_grouped_lookup_equals_the_oracle(s, S, k, nbytes, n):
    bf = _bf()
    block = s * S // 8
    nb = nbytes // block
    params = dict(num_blocks=nb, words_per_block=s, word_bits=S, k=k, seed=nb)
    words = _dense_words(nb * block, s + S)
    keys = _keys(n, "uniform", n)
    log(f"grouped lookup s={s} S={S} k={k} {nb * block} bytes, {n} keys")
    f = bf.BloomFilter(**params)
    try:
        f.load_words(torch.from_numpy(words).to("cuda"))
        out = torch.full((n + 16,), 7, dtype=torch.uint8, device="cuda")
        f.contains(to_device(keys), out=out[:n])
        got = out.cpu().numpy()
        want = oracle_par.contains(words, nb, s, S, k, nb, keys)
        assert np.array_equal(got[:n], want)
        assert (got[n:] == 7).all(), "results past the last key"
    finally:
        f.close()


@pytest.mark.parametrize("kind", ["repeated", "one"])
@pytest.mark.parametrize("nbytes,n", [(16 * MIB, (1 << 22) + 5), (96 * MIB, 12_000_007)])
def test_grouped_lookup_of_repeated_keys_and_odd_addresses(nbytes, n, kind):
    """Runs beyond their clip, keys 8 bytes and results 3 bytes into their
    buffers; a mapping of the caller's (one key at a time) gives the same."""
    bf = _bf()
    nb = nbytes // 32
    words = _dense_words(nbytes, 3)
    keys = _keys(n, kind, 9)
    log(f"grouped lookup, {kind} keys: {nbytes} bytes, {n} keys")
    f = bf.BloomFilter(nb, 8, 32, 8, 5)
    try:
        f.load_words(torch.from_numpy(words).to("cuda"))
        d = to_device(keys, offset_elems=1)
        out = torch.full((n + 32,), 7, dtype=torch.uint8, device="cuda")
        f.contains(d, out=out[3:n + 3])
        got = out.cpu().numpy()
        assert np.array_equal(got[3:n + 3], oracle_par.contains(words, nb, 8, 32, 8, 5, keys))
        assert (got[:3] == 7).all() and (got[n + 3:] == 7).all()
        f.set_mapping(bf.BF_OP_CONTAINS, 1, 8, 1)
        assert torch.equal(f.contains(d), out[3:n + 3])
    finally:
        f.close()


def test_grouped_lookup_of_a_parquet_filter():
    bf = _bf()
    nbytes, n = 32 * MIB, 5_000_001
    words = _dense_words(nbytes, 12)
    keys = _keys(n, "uniform", 13)
    log(f"grouped lookup, Parquet: {nbytes} bytes, {n} keys")
    f = bf.ParquetFilter(nbytes)
    try:
        f.load_words(torch.from_numpy(words).to("cuda"))
        got = f.contains(to_device(keys)).cpu().numpy()
        assert np.array_equal(got, oracle_par.parquet_contains(words, nbytes, keys))
    finally:
        f.close()


def test_large_lookup_in_a_captured_graph():
    """Captured, a large lookup allocates nothing and is replayed with eager
    lookups between the replays."""
    bf = _bf()
    n, nb = (1 << 22) + 123, 16 * MIB // 32
    f = bf.BloomFilter(nb, 8, 32, 8, 1)
    try:
        f.load_words(torch.from_numpy(_dense_words(nb * 32, 4)).to("cuda"))
        keys = to_device(_keys(n, "uniform", 21))
        want = f.contains(keys)
        out = torch.zeros(n, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            f.contains(keys, out=out)
        for replay in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want), f"replay {replay}"
            assert torch.equal(f.contains(keys), want)
    finally:
        f.close()


@pytest.mark.parametrize("kind", ["uniform", "repeated", "one"])
@pytest.mark.parametrize("chunks", [1, 5, 300, 1024, 1026, 2500])
def test_partitioned_add_at_step_edges(chunks, kind):
    """Key counts around a step, into filters of one digit (runs read by units
    of 16 and of 8 slots) and of two, each add on top of the last."""
    bf = _bf()
    nb = chunks * 2048 - (37 if chunks > 1 else 0)
    params = dict(num_blocks=nb, words_per_block=8, word_bits=32, k=8, seed=chunks)
    ref = oracle.OracleFilter(**params)
    f = bf.BloomFilter(**params)
    try:
        f.set_mapping(bf.BF_OP_ADD, strategy=bf.BF_STRATEGY_PARTITIONED)
        for i, n in enumerate((1, STEP - 1, STEP, STEP + 1, 9 * STEP + 17, 40 * STEP - 3)):
            keys = _keys(n, kind, 100 * chunks + i)
            log(f"partitioned add, {kind} keys: {chunks} chunks, {n} keys")
            f.add(to_device(keys))
            ref.add(keys)
            assert np.array_equal(f.words().cpu().numpy(), ref.bytes), f"{n} keys"
    finally:
        f.close()


@pytest.mark.parametrize("kind", ["uniform", "repeated"])
@pytest.mark.parametrize("gib", [4, 9, 17])
def test_partitioned_add_into_large_filters(gib, kind):
    """256 first digits and more: the second pass in units of 8 slots, with
    256, 512 and 1,024 second digits.  The words equal those of direct adds,
    which the oracle pins elsewhere; sampled blocks against the oracle."""
    bf = _bf()
    nb, n = (gib << 30) // 32 - 1001, (1 << 22) + 77
    keys = _keys(n, kind, gib)
    if kind == "repeated":  # direct adds of one key one after another are slow
        keys[keys == 77] = np.arange(int((keys == 77).sum()), dtype=np.uint64) % 4096
        keys[keys == 2**63] = np.arange(int((keys == 2**63).sum()), dtype=np.uint64) % 512
    log(f"partitioned add, {kind} keys: {gib} GiB, {n} keys")
    d = to_device(keys)
    f, g = bf.BloomFilter(nb, 8, 32, 8, 5), bf.BloomFilter(nb, 8, 32, 8, 5)
    try:
        f.set_mapping(bf.BF_OP_ADD, strategy=bf.BF_STRATEGY_PARTITIONED)
        g.set_mapping(bf.BF_OP_ADD, strategy=bf.BF_STRATEGY_DIRECT)
        f.add(d)
        g.add(d)
        words = f.words()
        assert torch.equal(words.view(torch.int64), g.words().view(torch.int64))
        sel = workloads.rng(gib).choice(nb, size=256, replace=False).astype(np.uint64)
        got = words.view(nb, 32)[torch.from_numpy(sel.astype(np.int64)).to("cuda")].cpu().numpy()
        assert np.array_equal(got, oracle.block_words(nb, 8, 32, 8, 5, keys, sel))
    finally:
        f.close()
        g.close()
