"""Host-side checks of bench.py that need no GPU: one partition on one GPU is all this build runs, so a
request for more GPUs must be refused with a message instead of being run on one."""
import ctypes as C
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_kernel_source_hash_covers_every_kernel_source():
    """The hash that ties a committed traffic profile to the build changes with any kernel source."""
    sys.path.insert(0, ROOT)
    import bench
    h = bench.kernel_source_hash()
    assert len(h) == 16 and int(h, 16) >= 0
    assert h == bench.kernel_source_hash()


@pytest.mark.parametrize("n_in,d_in,d_out", [(3073, 128, 112), (3073, 128, 113), (3072, 128, 47), (306250, 128, 47), (3073, 8, 7), (3073, 47, 128), (3073, 64, 64)])
def test_width_of_a_mean_aggregators_backward_pass_is_the_librarys(n_in, d_in, d_out):
    """The roofline's bytes count the width that is gathered.  The library shows it in the workspace: a second layer that gathers its output's gradient keeps
    a row of it per boundary node."""
    sys.path.insert(0, ROOT)
    import bench
    import paper_2203_10983_amd as pkg
    from test_abi import _descs
    size = []
    for n_halo in (1_000_000, 2_000_000):
        for dims in ((d_in, d_in, d_out), (d_in, d_in, d_in)):
            pd, md, keep = _descs(pkg, n_in=n_in, nnz0=n_in, e_in=n_in, n_halo=n_halo, dims=dims)
            md.layer_kind = 1
            size.append(pkg.load_library().bns_workspace_bytes(C.byref(pd), C.byref(md)))
    per_node = ((size[2] - size[0]) - (size[3] - size[1])) / 1_000_000
    width = bench.backward_width(d_in, d_out, 1, n_in)
    assert width in (d_in, d_out) and bench.backward_width(d_in, d_out, 0, n_in) == min(d_in, d_out)
    assert per_node == pytest.approx(4 * d_out if width < d_in else 0, abs=1)
