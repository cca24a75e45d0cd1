"""Tuned configurations keep the limits of the forms: the FP32 register tiles of the eight-product form, which do not flush their
sums, are neither kept by the autotuner nor loaded from a file for products of more than 2048 k."""
import numpy as np
import pytest

from conftest import rel_fro, to_dev, to_np
from oracle import quat as Q

pytestmark = pytest.mark.gpu


def _entries(text):
    return [tuple(line.split()[1:]) for line in text.splitlines() if line.startswith("gemm ")]


@pytest.mark.parametrize("m,n", [(20, 2500), (2049, 17)])
def test_autotuned_fp32_solve_flushes_long_sums(tmp_path, m, n):
    import paper_2605_01464_amd as q

    A = np.random.default_rng(m).standard_normal((4, m, n)).astype(np.float32).astype(np.float64)
    with q.Context(0) as c:
        c.set("autotune", 1)
        X, info = q.solve(c, to_dev(A, "f32"), "ns", tol=1e-6, precision="f32")
        c.save_tuning(tmp_path / "tune.txt")
    entries = _entries((tmp_path / "tune.txt").read_text())
    long = [name for p, _, _, k, name in entries if p == "1" and int(k) > 2048]
    assert long and "f32x8_16x16_regs4" not in long
    assert any("x8_" in name for name in long)
    assert rel_fro(to_np(X), Q.pinv_svd(A)) <= 1e-5


def test_tune_file_beyond_a_form_is_skipped(tmp_path):
    import paper_2605_01464_amd as q

    with q.Context(0) as c:
        q.qpinv_autotune(c.handle, q.GEMM_PREC["f32"], 40, 40, 40)
        c.save_tuning(tmp_path / "a.txt")
        head = (tmp_path / "a.txt").read_text().splitlines()[0]
        (tmp_path / "b.txt").write_text(head + "\ngemm 1 20 20 2048 f32x8_16x16_regs4\ngemm 1 20 20 2049 f32x8_16x16_regs4\n"
                                        "gemm 0 20 20 5000 f64x8_16x16_regs4\ngemm 1 24001 24001 64 f32_32x32x16_w2x2_mfma16_db\n")
        assert c.load_tuning(tmp_path / "b.txt") == 2
        c.save_tuning(tmp_path / "c.txt")
        kept = _entries((tmp_path / "c.txt").read_text())
    assert ("1", "20", "20", "2048", "f32x8_16x16_regs4") in kept and ("0", "20", "20", "5000", "f64x8_16x16_regs4") in kept
    assert len(kept) == 3


def _krylov_names(q, c, n, m):
    """Configurations of the n x m x n products of a Krylov run."""
    A = 3.0 * np.eye(n)[None] * np.array([1.0, 0, 0, 0]).reshape(4, 1, 1) + np.random.default_rng(1).standard_normal((4, n, n)) / n
    B = np.random.default_rng(2).standard_normal((4, n, m))
    c.set("gemm_timing", 1)
    q.qpinv_gemm_stats(c.handle)
    q.gl_krylov(c, to_dev(A, "f64"), to_dev(B, "f64"), tol=0.0, max_iter=3)
    _, rows = q.qpinv_gemm_stats(c.handle)
    c.set("gemm_timing", 0)
    return {q.qpinv_tile_config_name(r["prec"], r["cfg"]) for r in rows}


def test_tuned_choice_of_few_columns_is_used(tmp_path):
    import paper_2605_01464_amd as q

    with q.Context(0) as c:
        cfg, ms = q.qpinv_autotune(c.handle, q.GEMM_PREC["f64"], 100, 3, 100)
        name = q.qpinv_tile_config_name(q.GEMM_PREC["f64"], cfg)
        assert name and ms > 0.0
        assert _krylov_names(q, c, 100, 3) == {name}
        assert c.save_tuning(tmp_path / "a.txt") == 1
        text = (tmp_path / "a.txt").read_text()
        assert f"gemm 0 100 3 100 {name}" in text.splitlines()
        A, B = np.random.default_rng(3).standard_normal((2, 4, 100, 100))
        Ad, Bd = to_dev(A, "f64"), to_dev(B[:, :, :3], "f64")
        C = q.qgemm(c, Ad, Bd, cfg=cfg)
        assert rel_fro(to_np(C), Q.qmul(A, B[:, :, :3])) <= 1e-14
        head = text.splitlines()[0]
        for line, applied, used in (("gemm 0 100 3 100 f64_64x64x8_w4x4_mfma16", 1, "f64_64x64x8_w4x4_mfma16"),
                                    ("gemm 0 100 3 100 f64_16x16_narrow", 1, "f64_16x16_narrow"),
                                    ("gemm 0 100 17 100 f64_16x16_narrow", 0, "f64_16x16_narrow")):
            (tmp_path / "b.txt").write_text(head + "\n" + line + "\n")
            assert c.load_tuning(tmp_path / "b.txt") == applied
            assert _krylov_names(q, c, 100, 3) == {used}
