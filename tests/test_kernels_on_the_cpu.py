"""GPU tests with the kernels compiled for the CPU, where the wavefronts of a workgroup can be made to run far apart between
two barriers (on the GPU they nearly always run close together) and an access outside an allocation of device memory is
caught: behind its end where the wavefronts run in their order, before its start where they run in any order.  An access that
leaves a lane's or a channel's part of an allocation, or an array in LDS, for what lies beside it is not."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "emulated"))


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    import emulated_gpu
    return emulated_gpu.build(str(tmp_path_factory.mktemp("emulated")))


@pytest.mark.parametrize("any_order", [False, True])
@pytest.mark.parametrize("what", [
    # light frames that fill one of their structures: kept, or given up and redone in another form
    ["test_gpu_light_frame.py"],
    # states that meet in one slot of the table
    ["test_gpu_state_table.py"],
    # teams: the second call of a decoder starts with the histograms that the first one left
    ["test_gpu_random_sweep.py", "-k", "test_random_heavy_frames and (0] or 4])"],
])
def test_kernels_on_the_cpu(library, what, any_order):
    env = dict(os.environ, EMULATED_LIBRARY=library, PYTHONPATH=os.pathsep.join([os.path.dirname(HERE), os.path.join(HERE, "emulated")]))
    env.pop("EMULATED_ORDER", None)
    if any_order:
        env["EMULATED_ORDER"] = "1"
    run = subprocess.run([sys.executable, "-m", "pytest", "-q", "-x", "-p", "emulated_gpu", "-p", "no:cacheprovider", "-m", "gpu",
                          os.path.join(HERE, what[0])] + what[1:], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert run.returncode == 0, run.stdout[-3000:]


@pytest.mark.parametrize("states,bits", [(1, 4), (16, 4), (1536, 11), (2048, 11), (3072, 12)])     # to three quarters, and full
def test_what_is_put_into_a_state_table_is_found(library, states, bits, tmp_path):
    import emulated_gpu
    folder, program = os.path.dirname(library), str(tmp_path / "state_table")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-I" + emulated_gpu.HERE, "-I" + os.path.join(folder, "package", "csrc"),
                           os.path.join(emulated_gpu.HERE, "state_table.cpp"), os.path.join(emulated_gpu.HERE, "workgroup.cpp"), "-o", program, "-lpthread"])
    assert subprocess.run([program, str(states), str(bits)]).returncode == 0
