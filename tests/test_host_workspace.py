"""The selection's workspace size never falls with the number of segments: one workspace, sized for the
largest network, serves every smaller one."""
from paper_2109_00170_amd import _binding


def test_workspace_size_does_not_fall():
    size = _binding.load_library().alcs_select_workspace_bytes
    counts = list(range(0, 1100)) + [2000, 4096, 65535]
    sizes = [int(size(n)) for n in counts]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
    assert size(-1) == 0
