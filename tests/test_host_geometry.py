"""Launch geometry of the scoring passes, taken from the host side of the library built with a plain C++
compiler (kernel launchers replaced by stand-ins that note the geometry)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2605_06221_amd as up
from geometry_cases import HEAD_64

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST_BUILD = os.path.join(ROOT, "tests", "host_build")
CSRC = os.path.join(ROOT, "paper_2605_06221_amd", "csrc")


@pytest.fixture(scope="module")
def host_lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    lib = str(tmp_path_factory.mktemp("host") / "libuniprefill_host.so")
    cmd = [gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-x", "c++", "-I", HOST_BUILD, "-I", CSRC,
           os.path.join(CSRC, "up_api.hip"), os.path.join(HOST_BUILD, "launch_stubs.cpp"), "-o", lib]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    return ctypes.CDLL(lib)


def geometry(lib, lengths, num_q_heads, num_kv_heads, n_obs, head_dim=64, earlier=None, qk_dtype=up.UP_BF16, less=0):
    """((keys per work-group, split) of pass 1, the same of pass 2) of a score call given `less` bytes fewer than planned,
    and the planned workspace bytes; None where the call finds its workspace too small."""
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    cu_k = None if earlier is None else np.concatenate([[0], np.cumsum(np.add(lengths, earlier))]).astype(np.int32)
    ratio = np.full(len(lengths), 0.5, np.float32)
    p = up.make_params(num_seqs=len(lengths), total_tokens=int(cu[-1]), block_size=64, n_obs=n_obs, num_q_heads=num_q_heads,
                       num_kv_heads=num_kv_heads, head_dim=head_dim, hidden_dim=64, qk_dtype=qk_dtype)
    host = lambda a: ctypes.c_void_p(a.ctypes.data)
    dev = ctypes.c_void_p(1 << 20)          # never read: the launchers are stand-ins
    ws = ctypes.c_size_t(0)
    if earlier is None:
        assert lib.uniprefill_plan(ctypes.byref(p), host(cu), host(ratio), None, None, ctypes.byref(ws)) == 0
        room = ctypes.c_size_t(ws.value - less)
        st = lib.uniprefill_score(ctypes.byref(p), dev, dev, dev, host(cu), dev, dev, room, None)
    else:
        assert lib.uniprefill_plan_chunked(ctypes.byref(p), host(cu), host(cu_k), host(ratio), None, None, ctypes.byref(ws)) == 0
        room = ctypes.c_size_t(ws.value - less)
        st = lib.uniprefill_score_chunked(ctypes.byref(p), dev, dev, dev, host(cu), dev, host(cu_k), dev, dev, room, None)
    if st == up.UP_ERR_WORKSPACE:
        return None
    assert st == 0
    g = (ctypes.c_int32 * 4)()
    lib.stub_last_geometry(g)
    return (g[0], g[1]), (g[2], g[3]), ws.value


@pytest.mark.parametrize("name", HEAD_64)
def test_batches_of_the_gpu_tests_reach_their_geometry(host_lib, name):
    batch, pass1, pass2 = HEAD_64[name]
    assert geometry(host_lib, **batch)[:2] == (pass1, pass2)


@pytest.mark.parametrize("heads,window,lengths,key_block2", [
    ((32, 8), 128, [32768], 512), ((40, 8), 128, [30000], 512), ((32, 8), 128, [30000, 30000], 512),      # one round: as pass 1
    ((32, 8), 512, [122000], 512), ((32, 8), 128, [122000], 256), ((32, 8), 128, [131072], 256),
    ((32, 8), 128, [12289, 24576, 7011], 256), ((32, 8), 128, [1] * 64 + [28000, 100], 256), ((32, 8), 128, [8192] * 16, 256)])
def test_head_64_keeps_512_keys_where_one_round_of_them_is_faster(host_lib, heads, window, lengths, key_block2):
    (kb1, split1), (kb2, split2), _ = geometry(host_lib, lengths, *heads, window)
    assert kb1 == 512 and split2 == split1 and kb2 == key_block2


def test_other_head_rows_take_pass_1s_key_block_in_both_passes(host_lib):
    for lengths in ([32768], [131072], [12289, 24576, 7011], [4096], [1] * 64 + [28000, 100]):
        for head_dim, dtype in ((128, up.UP_BF16), (256, up.UP_BF16), (64, up.UP_F32), (128, up.UP_F32)):
            g1, g2, _ = geometry(host_lib, lengths, 32, 8, 128, head_dim=head_dim, qk_dtype=dtype)
            assert g1 == g2 and (g1[0] == 256 or (head_dim == 128 and dtype == up.UP_BF16))


def test_workspace_of_the_256_key_form_is_still_enough_where_512_keys_are_faster(host_lib):
    """The partial column sums of 116002 tokens in two sequences take 228 * 512 doubles or 455 * 256."""
    batch, pass1, pass2 = HEAD_64["whole_one_round_long_window"]
    assert geometry(host_lib, **batch)[1] == (512, 1)
    assert geometry(host_lib, **batch, less=2048)[1] == (256, 1)
    assert geometry(host_lib, **batch, less=2048 + 256) is None
    # nothing else has a smaller form
    for name in ("whole_many_rounds", "context"):
        assert geometry(host_lib, **HEAD_64[name][0], less=256) is None


def test_static_scratch_takes_what_fits_at_256_keys(host_lib):
    """A batch that needs 32 MiB + 2816 bytes at 512 keys and less than 32 MiB at 256 is not refused for its size (this
    build has no device: the call ends there)."""
    lengths = [19800] * 6
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ratio = np.full(6, 0.5, np.float32)
    assert geometry(host_lib, lengths, 32, 1, 521)[2] == up.STATIC_SCRATCH_BYTES + 2816
    p = up.make_params(num_seqs=6, total_tokens=int(cu[-1]), block_size=64, n_obs=521, num_q_heads=32, num_kv_heads=1,
                       head_dim=64, hidden_dim=64)
    host, dev = (lambda a: ctypes.c_void_p(a.ctypes.data)), ctypes.c_void_p(1 << 20)
    call = lambda: host_lib.uniprefill_fused_static(ctypes.byref(p), dev, dev, dev, dev, dev, host(cu), dev, host(ratio), dev, dev,
                                                    dev, dev, None, None)
    assert call() == up.UP_ERR_HIP
    p.n_obs = 523                     # too large in either form
    assert call() == up.UP_ERR_SCRATCH
