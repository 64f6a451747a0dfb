"""Where stage 4 takes the form with 64-bit offsets: a row of S_cq is 128 bytes, a listed token's number 32 bits."""
import os
import shutil
import subprocess

import pytest

from test_build_properties import CSRC, HIPCC, ROOT

CLAIMS = ["!plaid_wide(1, 0)", "!plaid_wide(1ll << 25, 1)", "plaid_wide((1ll << 25) + 1, 1)", "!plaid_wide(1, 1ll << 32)",
          "plaid_wide(1, (1ll << 32) + 1)", "!plaid_wide(262144, 600000000)"]


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_wide_form(tmp_path):
    unit = tmp_path / "rules.hip"
    unit.write_text('#include "plaid_internal.h"\n' + "".join(f'static_assert({c}, "{c}");\n' for c in CLAIMS))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                        "--cuda-host-only", "-fsyntax-only", str(unit)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
