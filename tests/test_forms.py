"""Rules that choose between forms of a kernel: the library's own host code, no GPU call."""
import shutil

import pytest

from test_host_logic import _run_host_program


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_forms_of_calls(tmp_path):
    _run_host_program("forms.hip", tmp_path, "--offload-arch=gfx950")
