"""The device check of canonical CSR over its entry tiles (3072 entries): faults
at the edges of tiles and of threads' stretches, in rows that cross tiles, in
tiles of more rows than mark their entries, and several at once; the flags named
in the error are those of a row-by-row walk on the host."""
import numpy as np
import pytest

import paper_2608_09713_amd as sp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    return torch.device("cuda:0")


def _csr(dev, rp, ci, n):
    import torch
    return sp.DeviceCSR(len(rp) - 1, n, torch.tensor(rp, dtype=torch.int64, device=dev),
                        torch.tensor(ci, dtype=torch.int32, device=dev),
                        torch.ones(len(ci), dtype=torch.float64, device=dev), int(rp[-1]))


def _rows(kind, rng):
    """row pointers and strictly increasing columns of a lower-triangular matrix"""
    if kind == "long":      # rows of 1 to 4000 entries, so tiles of one row and of a few
        lens = np.concatenate([np.arange(4000) % 5, [4000, 1, 3100, 3072, 2, 6144 // 2]])
    elif kind == "short":   # rows of up to two entries: over a thousand per tile
        lens = rng.integers(0, 3, 12000)
    else:                   # more rows in a tile than mark their entries
        lens = np.where(np.arange(60000) % 20 == 7, 1, 0)
    m = len(lens)
    lens = np.minimum(lens, np.arange(m) + 1)
    rp = np.zeros(m + 1, dtype=np.int64)
    rp[1:] = np.cumsum(lens)
    ci = np.concatenate([np.sort(rng.choice(i + 1, size=n, replace=False)) for i, n in enumerate(lens) if n])
    return rp, ci.astype(np.int64), m


def _flags(rp, ci, n, lower):
    row = np.repeat(np.arange(len(rp) - 1), np.diff(rp))
    first = np.zeros(len(ci), dtype=bool)
    first[rp[:-1][np.diff(rp) > 0]] = True
    return {"column-range": bool(((ci < 0) | (ci >= n)).any()),
            "column-order": bool((~first[1:] & (ci[:-1] >= ci[1:])).any()),
            "above-diagonal": bool(lower and (ci > row).any())}


@pytest.mark.parametrize("kind", ["long", "short", "sparse"])
def test_validation_flags(dev, kind):
    rng = np.random.default_rng(3)
    rp, ci, m = _rows(kind, rng)
    nnz = len(ci)
    assert nnz > 2900
    sp.mirror(_csr(dev, rp, ci, m), "f64")  # accepted as it is
    inner = np.flatnonzero(np.repeat(np.diff(rp), np.diff(rp)) > 1)
    inner = inner[~np.isin(inner, rp)]  # entries with a predecessor in their row
    at = [p for p in (0, 11, 12, 3071, 3072, 3083, 6143, 6144, nnz - 1) if p < nnz]
    at += [int(p) for p in rng.choice(inner, 4)] if len(inner) else []
    for p in at:
        row = int(np.searchsorted(rp, p, side="right") - 1)
        for what, value in (("past", m), ("negative", -1), ("repeat", ci[p - 1] if p else 0),
                            ("above", min(m - 1, row + 1))):
            bad = ci.copy()
            bad[p] = value
            want = _flags(rp, bad, m, True)
            print(f"[validate tiles] {kind} entry {p} {what} {want}", flush=True)
            if not any(want.values()):
                continue
            with pytest.raises(sp.SpsyrkError) as e:
                sp.mirror(_csr(dev, rp, bad, m), "f64")
            assert {k: k in str(e.value) for k in want} == want
