"""CPU-only checks of the boundary: the library loads and exports every symbol
the header declares; the binding refuses to run without a GPU (no fallback)."""

import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "artopk.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(artopk_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported():
    import paper_2312_02493_amd as pkg

    names = _declared_symbols()
    assert {"artopk_variance", "artopk_select_topk", "artopk_gather_sum", "artopk_scatter_residual",
            "artopk_step", "artopk_create", "artopk_destroy"} <= set(names)
    lib = pkg.load_library()
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(pkg.exported_symbols()) == names
    assert lib.artopk_version() >= 100


def test_scratch_size_query():
    """artopk_scratch_bytes is host arithmetic: the size of the one allocation artopk_create makes.
    Checked against the terms the header's comment on artopk_create lists (dominant ones only, so
    within a few percent), its monotonicity in every limit, and the limits artopk_create refuses."""
    import paper_2312_02493_amd as pkg

    q = pkg.artopk_scratch_bytes
    n, w, k = 1_000_000_000, 8, 1_000_000
    got = q(w, n, k, 1)
    model = (w * 16.4 * 2**20            # per-chunk histograms and the rest of a worker's slot
             + 8 * (k + max(n // 8, 2**22))  # survivor list
             + 8 * w * k                  # value rows and index rows
             + w * n / 8                  # bit masks
             + 1.5 * n)                   # staged list entries
    assert abs(got - model) / model < 0.03, (got, model)
    assert 3.5e9 < got < 4.0e9           # the figure the design notes quote for this size
    for w, n, k in ((1, 1 << 16, 100), (1, 1 << 20, 10_000), (8, 1 << 20, 10_000), (16, 1 << 18, 2_000),
                    (64, 1 << 21, 20_000), (8, 11_689_512, 116_896), (8, 1_000_000_000, 1_000_000)):
        batch = min(w, 16)
        model = (w * 16.4 * 2**20 + 64 * 2**10 * batch + 8 * min(n, k + max(n // 8, 2**22)) + 8 * w * k + w * n / 8
                 + 1.5 * n + batch * n / 341 + w * 128 * 2**10 + 4.5 * min(n, 2**21) + 1.25 * 2**20)
        assert abs(q(w, n, k, 1) - model) / model < 0.015, (w, n, k, q(w, n, k, 1), model)
    n, w, k = 1_000_000_000, 8, 1_000_000
    assert q(w, n, k, 1) <= q(w + 1, n, k, 1) and q(w, n, k, 1) <= q(w, n, k * 2, 1) and q(w, n, k, 1) <= q(w, n, k, 9)
    assert q(w, 1 << 20, 1024, 1) < q(w, 1 << 24, 1024, 1)
    assert q(1, 1, 1, 1) > 0
    for bad in ((0, 10, 1, 1), (65, 10, 1, 1), (1, 0, 1, 1), (1, 1 << 31, 1, 1), (1, 10, 0, 1), (1, 10, 11, 1),
                (1, 10, 1, 0), (1, 10, 1, 65536)):
        assert q(*bad) == -1, bad


def test_no_cpu_fallback():
    import torch
    import paper_2312_02493_amd as pkg

    if torch.cuda.is_available():
        pytest.skip("GPU present")
    with pytest.raises(RuntimeError):
        pkg.Context(2, 1024, 16)


def test_product_does_not_import_oracle():
    pkg_dir = os.path.join(ROOT, "paper_2312_02493_amd")
    for dirpath, _, files in os.walk(pkg_dir):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                src = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in src.lower(), f
