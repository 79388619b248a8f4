"""The machine code around the LDS loads of the wide products and of those with few tokens, under the same rules as that of
the output tiles; and the stores that the waits of the wide ones count on."""
import os

import pytest
import test_generated_code as rules

from paper_2309_03824_amd import build


@pytest.fixture(scope="module", params=[("mfma_wide", 32), ("mfma_small", 5)], ids=lambda p: p[0])
def kernels(request, tmp_path_factory):
    name, count = request.param
    obj = os.path.join(build.OBJ, name + ".hip.o")
    if not os.path.exists(obj):
        os.makedirs(build.OBJ, exist_ok=True)
        build._compile(os.path.join(build.CSRC, name + ".hip"))
    patch = pytest.MonkeyPatch()
    patch.setattr(rules, "OBJ", obj)
    try:
        listing = rules.listing(tmp_path_factory.mktemp("code"))
        assert len(listing) == count
        return listing
    finally:
        patch.undo()


def test_descriptors_are_settled(kernels):
    assert not {k: [hex(a) for a in rules.faults(rows)] for k, rows in kernels.items() if rules.faults(rows)}


def test_m0_belongs_to_the_loads(kernels):
    # (the loads stand in loops: a few places in each kernel)
    loads = [sum(op.startswith("buffer_load") and args.endswith(" lds") for _, op, args, _ in rows) for rows in kernels.values()]
    assert min(loads) > 0 and rules.m0_writes(kernels) == sum(loads)


def test_nothing_is_spilled(kernels):
    assert not [k for k, rows in kernels.items() if any(op.startswith("scratch_") for _, op, _, _ in rows)]


def test_every_chunk_stores_without_a_branch(kernels):
    # a wave waits for "all but the newest 4 (with GELU 8)": that many stores follow the loads, whatever rows exist
    for k, rows in kernels.items():
        if "wide_kernel" not in k:
            continue
        n = 8 if "ELi1EEE" in k else 4
        stores = [i for i, r in enumerate(rows) if r[1] == "buffer_store_dwordx4"]
        targets = {r[3] for r in rows}
        assert stores and len(stores) % n == 0, k
        for first in range(0, len(stores), n):
            for i in range(stores[first], stores[first + n - 1]):
                assert rows[i][3] is None and rows[i + 1][0] not in targets, k
