"""The comparison switches TSM_IGEMM_RING=0 / TSM_WGRAD_TR=0 route the bf16 convolutions to the register-prefetch and
register-transposing kernels (the ones that otherwise serve channel counts that are not multiples of 64) and the
inference path to its unfused form.  The switches are read once per process, so a child process runs a few of the
parity tests under them."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_parity_holds_on_the_fallback_kernels():
    env = dict(os.environ, TSM_IGEMM_RING="0", TSM_WGRAD_TR="0")
    picks = ["tests/test_gpu_infer.py::test_infer_bf16_against_oracle",
             "tests/test_gpu_block.py::test_config1_bottleneck_reduced",
             "tests/test_gpu_block.py::test_bottleneck_projection_stride2",
             "tests/test_gpu_step.py::test_step_bf16_against_oracle_reduced_size"]
    r = subprocess.run([sys.executable, "-m", "pytest", "-q", "-x", "-m", "gpu", "-p", "no:cacheprovider"] + picks,
                       cwd=ROOT, env=env, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


CHILD = """
import json, sys
sys.path[:0] = [%r, %r]
import test_gpu_block, test_gpu_infer, test_gpu_step
from paper_1910_00932_amd import binding as B
out = {}
for name, f in (("block", lambda: test_gpu_block.run_block("bottleneck", 1, 4, 256, 14, 14, 128, 512, 2, True, 8, "bf16", "nthwc")),
                ("infer", test_gpu_infer.test_infer_bf16_against_oracle),
                ("step", test_gpu_step.test_step_bf16_against_oracle_reduced_size)):
    B.tsm_profile_begin()
    f()
    out[name] = sorted(B.tsm_profile_end())
    print(name, "done", flush=True)
print(json.dumps(out))
""" % (ROOT, os.path.join(ROOT, "tests"))


def test_the_switches_reach_the_fallback_kernels():
    """What ran in those tests, whose layers are all small: the register-prefetch kernels in both directions, no kernel for
    64-channel steps but the stem's, no K-split kernel, and inference with its BatchNorm passes."""
    env = dict(os.environ, TSM_IGEMM_RING="0", TSM_WGRAD_TR="0")
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=env, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    ran = {k: set(v) for k, v in json.loads(r.stdout.splitlines()[-1]).items()}
    print(ran)
    both = {"igemm_fwd_128x128", "igemm_dgrad_128x128"}
    assert both <= ran["block"] and both | {"igemm_fwd_128x64", "igemm_dgrad_128x64"} <= ran["step"], ran
    assert {"igemm_fwd_128x64", "igemm_fwd_128x128", "bn_relu_apply", "block_tail_fwd"} <= ran["infer"], ran
    general = lambda v: {k for k in v if k.startswith("igemm") and not k.split("_")[2].startswith("128x")}   # noqa: E731
    assert not general(ran["block"]) and len(general(ran["infer"])) == len(general(ran["step"])) == 1, ran
    assert not any("ksplit" in k or "fused_tail" in k for v in ran.values() for k in v), ran
