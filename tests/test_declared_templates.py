"""Function templates that are specialised in another translation unit are declared so wherever they are called: a call of a template without
a definition would otherwise instantiate it implicitly, and a specialisation that only another unit knows makes that ill-formed."""
import os
import subprocess

from paper_2604_04921_amd import build as B


def test_no_call_of_a_template_without_definition():
    res = subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "--offload-host-only", "-fsyntax-only", "-Werror=undefined-func-template", "-I",
                          os.path.join(B.ROOT, "include"), "-I", B.CSRC, os.path.join(B.CSRC, "tri_score.hip")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0, res.stdout
