"""The stored launch shapes hold what the autotuner sets for a context and
nothing else: an entry that stands for "not tuned" would pin the form it names,
where a context without it takes the form that is fastest at the level's size."""

import json

import pytest

import paper_1402_3545_amd as G


def _tables():
    with open(G.LAUNCH_TABLE) as fh:
        return sorted(json.load(fh).items())


@pytest.mark.parametrize("key,table", _tables())
def test_stored_tables_hold_tuned_entries_only(key, table):
    levels, prec = int(key.split("|")[2][1:]), key[-1]
    want = set()
    for lvl in range(levels):
        kinds = {"spmv", "residual", "line_solve", "smooth"}
        kinds |= {"residual_restrict", "prolong_smooth"} if lvl < levels - 1 else set()
        kinds |= {"prolongate"} if lvl else set()
        want |= {f"{k}/{lvl}/{prec}" for k in kinds}
    # the finest level's FP64 solver kernels
    want |= {f"{k}/0/0" for k in ("cg_spmv", "cg_tridiag", "fcg")}
    if prec == "1":
        want |= {"residual/0/0", "correct/0/0"}
    assert set(table) == want
    assert all(k.split("/")[0] in G.TUNED_KERNELS for k in table)
