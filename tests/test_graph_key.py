"""The captured iteration graphs of a batch hold the addresses of the solver's buffers: every device buffer of the
vector kernels is in the key a kept graph is found by, and none is cleared on the null stream, which the batch's
(non-blocking) streams do not wait for."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_02490_amd", "csrc")


def read(name):
    return open(os.path.join(CSRC, name)).read()


def test_buffers_of_the_vector_kernels_are_in_the_graph_key():
    struct = re.search(r"struct Blas \{(.*?)\n\};", read("blas.h"), flags=re.S).group(1)
    members = [m.strip() for line in re.findall(r"^\s*DevBuf ([^;]*);", struct, flags=re.M) for m in line.split(",")]
    assert "scal" in members
    batched = read("batched.hip")
    key = batched[batched.index("key = {"):batched.index("key.push_back(v)")]
    assert not [m for m in members if f"blas.{m}.p" not in key]


def test_no_clear_on_the_null_stream():
    assert not re.findall(r"\bhipMemset\(", read("blas.hip"))
