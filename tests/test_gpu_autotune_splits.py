"""Row splits that the autotuner times for the FP32 logistic step, and the file of
its choices: the split count that an untuned context uses is among them, the others
are ones that keep a split's chains on one XCD, and a file written for replaced
kernels is passed over.
"""
import os
import re
import subprocess
import sys

import pytest

import workloads as W
from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2002_01184_amd import hmc  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("N,D,C", [(6931, 12, 3691), (3000, 41, 200), (70, 40, 64), (40, 50, 64)])
def test_candidates(N, D, C):
    w = W.logreg(N, D, C, L=2, step_size=0.001, seed=1, init=0.1)
    s = hmc.sampler_for(w, form=hmc.HMC_FORM_PLAIN)
    splits = [int(v) for v in re.findall(r"lr_nsplit=(\d+) ", s.autotune(1))]
    s.close()
    print(f"{N}x{D}, {C} chains: splits {splits} (0: the untuned choice)")
    assert splits[0] == 0 and len(set(splits)) == len(splits)
    assert all(v <= 8 or v % 8 == 0 for v in splits)
    assert all(v <= max(1, -(-N // 64)) for v in splits)


def test_choices_for_replaced_kernels_are_passed_over(tmp_path):
    code = ("import workloads as W; from paper_2002_01184_amd import hmc; "
            "s = hmc.sampler_for(W.logreg(2100, 40, 64, L=2, step_size=0.001, seed=1, init=0.1), "
            "form=hmc.HMC_FORM_PLAIN); print('REPORT', s.autotune(1).splitlines()[0]); s.close()")
    path = tmp_path / "choices"
    path.write_text("3:40:11:6:1:1:2:1 1 3 0 0\n")            # as it was written before keys had a version
    env = dict(os.environ, HMC_AUTOTUNE_CACHE=str(path), PYTHONPATH=ROOT)
    first, second = (subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, check=True, timeout=60,
                                    capture_output=True, text=True).stdout for _ in range(2))
    assert "REPORT form=1" in first and "cached" not in first
    assert "REPORT cached" in second


def test_choice_of_the_fused_form_is_not_taken_where_it_does_not_fit(tmp_path):
    # 1024 and 1500 rows share a key; the fused logistic kernel ends at 1024
    code = ("import workloads as W; from paper_2002_01184_amd import hmc; "
            "s = hmc.sampler_for(W.logreg(1500, 25, 64, L=2, step_size=0.01, seed=1)); "
            "s.autotune(1); s.sample_chain(2, 0); print('FORM', s.form); s.close()")
    path = tmp_path / "choices"
    path.write_text("v2:3:25:10:6:1:1:2:0 2 0 0 0\n")
    env = dict(os.environ, HMC_AUTOTUNE_CACHE=str(path), PYTHONPATH=ROOT)
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, timeout=60, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    assert "FORM plain" in out.stdout or "FORM graph" in out.stdout
