"""Traffic records: the hash that decides whether bench.py still accepts a measured record
covers everything that the kernel is compiled from."""
import os
import re

import pytest

import profile_summary as P

ENTRIES = [(w, inst, files) for w, order in P.VARIANT_ORDERS.items() for inst, (_, files) in order.items()]


@pytest.mark.parametrize("workload,inst,files", ENTRIES)
def test_every_included_header_is_hashed(workload, inst, files):
    hashed = P.with_headers(files)
    for f in hashed:
        text = open(os.path.join(P.CSRC, f)).read()
        for h in re.findall(r'#include "([^"]+)"', text):
            assert os.path.basename(h) in hashed, (f, h)
    kernel = re.search(r"ins::(k_\w+)", inst).group(1)
    assert any(re.search(rf"void {kernel}\(", open(os.path.join(P.CSRC, f)).read()) for f in hashed), kernel


def test_a_changed_header_invalidates_a_record(tmp_path, monkeypatch):
    files = P.with_headers(["k_fft.hip"])
    assert "k_fft.hpp" in files and "k_common.hpp" in files
    for f in files:
        (tmp_path / f).write_text(open(os.path.join(P.CSRC, f)).read())
    before = P.source_hash(files)
    monkeypatch.setattr(P, "CSRC", str(tmp_path))
    assert P.source_hash(files) == before
    (tmp_path / "k_fft.hpp").write_text("// changed\n")
    assert P.source_hash(files) != before
