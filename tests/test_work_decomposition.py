"""Which launches group the workgroups of a subgraph on one XCD (host only, no device call)."""
import numpy as np
import pytest

from paper_2511_09261_amd import binding

KINDS = ("forward", "hidden", "embed")


def sizes(n, P, spread, seed):
    share = 1.0 + spread * (2.0 * np.random.RandomState(seed).random_sample(P) - 1.0)
    return np.diff(np.round(np.cumsum(np.append(0.0, share)) / share.sum() * n)).astype(np.int32)


def grouped(part):
    """Every subgraph's workgroups on one XCD (ids equal modulo 8), as opposed to consecutive ids."""
    ids = np.arange(part.size)
    one_xcd = all(np.unique(ids[part == k] % 8).size == 1 for k in np.unique(part[part >= 0]))
    in_order = bool((np.diff(part) >= 0).all())
    assert one_xcd != in_order
    return one_xcd


@pytest.mark.parametrize("seed", range(8))
def test_uneven_subgraphs_of_wide_fp32_rows_are_not_grouped(seed):
    """Grouped, these took 465 -> 566 us (width 64) and 466 -> 611 us (width 128) per epoch."""
    for n, dim, P in ((150_001, 64, 24), (150_001, 64, 48), (100_000, 128, 24)):
        rows = sizes(n, P, 0.5, seed)
        for kind in KINDS:
            assert not grouped(binding.workgroup_parts("fp32", dim, kind, rows, rows * 11))


@pytest.mark.parametrize("n,dim,P,spread", [(700_001, 16, 48, 0.3), (600_000, 16, 64, 0.0), (300_000, 32, 64, 0.0),
                                            (1_200_000, 8, 64, 0.0)])
def test_narrow_fp32_rows_beyond_the_caches_are_grouped_evenly(n, dim, P, spread):
    rows = sizes(n, P, spread, 1)
    for kind in KINDS:
        part = binding.workgroup_parts("fp32", dim, kind, rows, rows * 3)
        assert grouped(part)
        assert part.size * 100 <= (part >= 0).sum() * 105
        assert (np.bincount(part[part >= 0], minlength=P) > 0).all()


def test_what_is_never_grouped():
    one_giant = np.array([500_000] + [10_000] * 20, dtype=np.int32)      # an XCD would have most of the work
    few = np.array([100_000] * 7, dtype=np.int32)                        # fewer subgraphs than XCDs
    small = np.array([10_000] * 48, dtype=np.int32)                      # below 32 MB
    for rows, dim, storage in ((one_giant, 16, "fp32"), (few, 16, "fp32"), (small, 16, "fp32"),
                               (np.array([20_000] * 50, dtype=np.int32), 64, "bf16")):
        for kind in KINDS:
            assert not grouped(binding.workgroup_parts(storage, dim, kind, rows, rows * 3))
    with pytest.raises(binding.GcoError):
        binding.workgroup_parts("bf16", 16, "forward", few, few)
    with pytest.raises(binding.GcoError):
        binding.workgroup_parts("fp32", 16, "forward", [0], [4])
