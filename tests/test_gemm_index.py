"""Host test of the GEMM's operand addresses (csrc/gemm_index.hpp), compiled
with g++: every load of every planned kernel lies inside its operand, the
ones past a range's end too, and those that matter are at their values."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM_INC = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INC),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("gemm_index") / "gemm_index_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INC,
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2607_20214_amd", "csrc"),
                    os.path.join(HERE, "host", "gemm_index_check.cpp"), "-o", out], check=True)
    return out


def test_every_load_lies_inside_its_operand(exe):
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout + r.stderr


def plan(exe, M, N, K, ta, tb, heads=(0, 0, 0), seq=0):
    r = subprocess.run([exe, *map(str, (M, N, K, int(ta), int(tb), *heads, seq))], capture_output=True, text=True, check=True)
    kind, splits, kper = r.stdout.split()
    return kind, int(splits), int(kper)


def test_walk_reaches_a_last_split_of_less_than_a_k_tile(exe):
    """dW_O of a block of d_model 1024 over 13448 tokens: the large kernel's last split holds 8 values of k."""
    kind, splits, kper = plan(exe, 1024, 1024, 13448, 1, 0, (16, 0, 0), 13448)
    assert kind == "large" and 0 < 13448 - (splits - 1) * kper < 64


@pytest.mark.parametrize("M,N,K", [(8388608, 8388608, 8), (2147483640, 2147483640, 8), (2147483640, 8, 2147483640),
                                   (8, 8, 2147483640), (2147483640, 2147483640, 2147483640)])
def test_plan_of_any_size(exe, M, N, K):
    """A workspace query may name any sizes: tile counts past 2^31 (and 2^32
    exactly, which an int count held as 0 and divided by) are planned."""
    kind, splits, kper = plan(exe, M, N, K, 0, 0)
    assert kper > 0 and kper % 64 == 0 and 0 <= (splits - 1) * kper < K <= splits * kper


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("seq,nseq", [(262144, 1), (262144, 3), (2097152, 1)])
def test_large_head_major_products_keep_the_large_kernel(exe, seq, nseq, dh):
    """O W_O, dQKV W_QKV', dW_O and dW_QKV of d_model 2048 over sequences whose
    rows of all heads are past 2^31 bytes: no tile spans them."""
    n, dm, H = seq * nseq, 2048, 2048 // dh
    for shape, ta, tb, heads in [((n, dm, dm), 0, 0, (H, 0, 0)), ((n, dm, 3 * dm), 0, 1, (3 * H, 0, 0)),
                                 ((dm, dm, n), 1, 0, (H, 0, 0)), ((dm, 3 * dm, n), 1, 0, (0, 3 * H, 0))]:
        assert plan(exe, *shape, ta, tb, heads, seq)[0] == "large", (shape, heads)
