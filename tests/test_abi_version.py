"""A library of another ABI version is refused with the advice to rebuild it, whatever entry points it
lacks; the binding and the header name the same version."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_binding_and_header_agree():
    from paper_2002_00250_amd import fgs
    text = open(os.path.join(ROOT, "include", "fgs.h")).read()
    assert int(re.search(r"#define FGS_ABI_VERSION (\d+)", text).group(1)) == fgs.ABI_VERSION
    # the entry points that came with version 7
    assert fgs.ABI_VERSION >= 7 and all(hasattr(fgs.lib(), n) for n in (
        "fgs_push_frame_on", "fgs_get_mask_on", "fgs_eval_accumulate_on", "fgs_order_create", "fgs_window_bce",
        "fgs_window_bce_keep", "fgs_window_bce_kept_grad"))


@pytest.mark.parametrize("source", ["int fgs_abi_version(void) { return 6; }", "int nothing;"])
def test_another_version_is_refused(tmp_path, monkeypatch, source):
    from paper_2002_00250_amd import fgs
    src, lib = tmp_path / "old.c", tmp_path / "libold.so"
    src.write_text(source + "\n")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    monkeypatch.setattr(fgs, "LIB_PATH", str(lib))
    monkeypatch.setattr(fgs, "_lib", None)
    with pytest.raises(fgs.FgsError) as e:
        fgs.lib()
    assert "rebuild" in str(e.value)
