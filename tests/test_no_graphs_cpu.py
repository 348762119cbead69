"""The library makes no HIP graph: the classes of a batched call were the nodes of
one once, and the host process crashed inside that call, with the graph calls as
the only suspects left."""
import subprocess

from paper_2203_10213_amd import vkt


def test_library_calls_no_graph_function():
    names = subprocess.run(["nm", "-D", "--undefined-only", vkt.LIB_PATH], capture_output=True,
                           text=True, check=True).stdout.split()
    assert any(n.startswith("hipLaunchKernel") for n in names)
    assert not [n for n in names if n.startswith("hipGraph")]
