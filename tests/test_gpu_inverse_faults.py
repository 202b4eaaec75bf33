"""Blocks without an inverse in a batch of good ones, in every kernel shape of the inverse:
singular ones, and ones that hold a NaN or an infinity, are reported and the others
inverted."""
import functools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


def zero_row_and_column(M, d):
    M[:, d // 2] = 0.0
    M[d // 2, :] = 0.0


def equal_rows(M, d):
    M[d - 1] = 0.0
    M[:, d - 1] = 0.0


def nan_entry(M, d):
    M[d // 3, d - 1] = np.nan


def nan_imaginary(M, d):
    M[d - 1, 0] = complex(1.0, np.nan)


def inf_entry(M, d):
    M[0, d // 2] = np.inf


def minus_inf_imaginary(M, d):
    M[d // 2, d // 2] = complex(0.5, -np.inf)


@functools.lru_cache(maxsize=None)
def problem(d):
    rng = np.random.default_rng(d)
    M = (rng.normal(size=(3, d, d)) + 1j * rng.normal(size=(3, d, d))) / np.sqrt(d) + np.eye(d)
    return M, [np.linalg.cond(x) for x in M]


@pytest.mark.parametrize("d", [20, 64, 100, 113, 128, 250, 500, 513, 700, 1024])
@pytest.mark.parametrize("spoil", [zero_row_and_column, equal_rows, nan_entry, nan_imaginary, inf_entry,
                                   minus_inf_imaginary])
def test_bad_block_is_reported_and_the_others_inverted(torch, d, spoil):
    from paper_2601_04904_amd.solver import diag_inverse
    good, cond = problem(d)
    M = good.copy()
    spoil(M[1], d)
    dst, bad = diag_inverse(torch.from_numpy(M).cuda())
    assert bad == 1
    for i in (0, 2):
        # 50 eps sqrt(d) cond, as the other inverse tests, on the residual
        got = dst[i].cpu().numpy()
        res = np.linalg.norm(good[i] @ got - np.eye(d)) / np.sqrt(d)
        assert res < 50 * 2.0 ** -52 * np.sqrt(d) * cond[i], (i, res)


@pytest.mark.parametrize("d", [20, 100, 200, 600])
def test_entries_whose_parts_add_up_past_the_range(torch, d):
    """|re| + |im| overflows while the entry and its reciprocal are finite."""
    from paper_2601_04904_amd.solver import diag_inverse
    rng = np.random.default_rng(d)
    v = np.where(rng.uniform(size=d) < 0.5, 1.2e308 + 1.1e308j, 1.0 - 2.0j)
    M = np.diag(v)[None][:, rng.permutation(d)]
    dst, bad = diag_inverse(torch.from_numpy(np.ascontiguousarray(M)).cuda())
    assert bad == -1
    got = dst[0].cpu().numpy() @ M[0]
    assert np.abs(got - np.eye(d)).max() < 1e-14
