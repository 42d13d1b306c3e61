"""What the library asks of the HIP runtime, in order (no GPU): hip_record.cpp defines
the runtime functions, runs calls of the C ABI and prints each request."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    """record(*commands): [(command, status, [request, ...]), ...]"""
    from paper_2204_13595_amd import irbe
    if not os.path.exists(irbe.LIB_PATH):
        from paper_2204_13595_amd import build
        build.build(verbose=False)
    exe = str(tmp_path_factory.mktemp("hip_record") / "hip_record")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{os.path.join(ROOT, 'include')}",
                    os.path.join(HERE, "hip_record.cpp"), "-rdynamic", "-ldl", "-o", exe], check=True)

    def run(*commands):
        r = subprocess.run([exe, irbe.LIB_PATH, *commands], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        calls, requests = [], []
        for line in r.stdout.splitlines():
            if line.startswith("= "):
                name, status = line[2:].rsplit(" ", 1)
                calls.append((name, int(status), requests))
                requests = []
            else:
                requests.append(line)
        assert [c[0] for c in calls] == list(commands)
        return calls

    return run


def _last(requests, *kinds):
    return max((i for i, r in enumerate(requests) if r.split()[0] in kinds), default=-1)


@pytest.mark.parametrize("types", [1, 4, 5])
def test_set_system_waits_for_its_copies(record, types):
    """The caller's arrays and the tables made on the host are free again on return."""
    (_, st0, _), (_, st1, requests) = record(f"create:n=100,types={types},mol=3", "set")
    assert st0 == st1 == 0
    assert _last(requests, "copy", "launch") > 0
    assert _last(requests, "wait") > _last(requests, "copy", "launch")


@pytest.mark.parametrize("types", [1, 4, 5])
def test_tables_are_refused_under_capture_before_anything_is_queued(record, types):
    """A wait or a pageable copy would invalidate the caller's capture."""
    calls = record(f"create:n=100,types={types}", "set", "capture=1", "lj", "capture=0", "lj")
    name, status, requests = calls[3]
    assert (status, requests) == (-6, [])
    assert calls[5][1] == 0 and _last(calls[5][2], "copy", "launch") >= 0


@pytest.mark.parametrize("n", [1, 2, 3, 7, 18, 30, 33, 95])
@pytest.mark.parametrize("hint", [0, 50, 1000])
def test_list_rows_are_whole_16_byte_units(record, n, hint):
    """The pair kernel and the list build take four entries at a time from the start
    of any row, so the capacities of small systems, which are bounded by the number
    of atoms, are multiples of four as well."""
    calls = record(f"create:n={n},box=9,hint={hint},entries=32", "set", "build", "counts")
    assert [c[1] for c in calls] == [0, 0, 0, 0]
    core, shell = (int(x) for x in calls[3][2][-1].split()[1:])
    assert core % 4 == 0 and shell % 4 == 0 and min(core, shell) >= min(n, 32)


def test_crowded_row_is_no_error(record):
    """A stencil row of many candidates (bit 3 of the error word) leaves the masks of that
    build whole: the handle takes 32-bit entries with the next build, and nothing fails."""
    calls = record("create:n=4000,box=4", "set", "build", "overflow=0,0,0,8", "build", "sync", "overflow=0,0,0,0",
                   "build", "sync")
    assert [c[1] for c in calls] == [0] * len(calls)
    masks = [any("k_list_blocks" in r and "ELb1ELb0EEE" in r for r in calls[i][2]) for i in (2, 4, 7)]
    assert masks == [True, True, False]


@pytest.mark.parametrize("n,box,rows,segments", [(600, 39.1, 49, 7), (1000, 46.4, 81, 3), (12000, 106.2, 441, 2)])
def test_dilute_rows_are_cut_where_a_window_ends(record, n, box, rows, segments):
    """The list build of few ions takes one wavefront per segment of a cell row that a
    window of the box allows, not one per row that takes them in turn."""
    calls = record(f"create:n={n},box={box},rcore=5,rshell=15", "set", "build")
    launch = [r.split() for r in calls[2][2] if "k_build_lists_lanes" in r]
    assert len(launch) == 1 and int(launch[0][2]) == rows * segments


@pytest.mark.parametrize("per_mol,by_id", [(3, False), (201, False), (202, True), (1000, True)])
def test_large_molecules_are_excluded_by_id(record, per_mol, by_id):
    """Up to 200 excluded partners are cleared from the masks one by one; for more the list
    build compares ids, and the partners' sorted indices take a launch of their own."""
    calls = record(f"create:n=4000,box=3.42,mol={per_mol}", "set", "build")
    names = [r.split()[1] for r in calls[2][2] if r.startswith("launch")]
    assert any("k_excl_sorted" in n for n in names) == by_id
    assert any("k_list_blocksILi0ELb0ELb1ELb%dEEE" % by_id in n or "k_list_blocksILi0ELb1ELb1ELb%dEEE" % by_id in n
               for n in names)


@pytest.mark.parametrize("k", [0, 1, 2])
def test_a_build_after_a_failed_growth_allocates_first(record, k):
    """Rows that a failed growth has given up are allocated before any kernel is queued."""
    calls = record("create:n=4000,box=4", "set", "build", "overflow=5000,100,0,2", "build", f"fail={k}", "sync",
                   "overflow=0,0,0,0", "forces", "fail=0", "build", "build", "forces")
    status = [c[1] for c in calls]
    assert status[:6] == [0] * 6 and status[6] == -2  # IRBE_ENOMEM
    assert status[8] == -5                            # forces: IRBE_ESTATE
    assert status[10] == -2 and not [r for r in calls[10][2] if r.startswith("launch")]
    assert status[11] == status[12] == 0
    assert [r for r in calls[11][2] if r.startswith("malloc")]


@pytest.mark.parametrize("n,p,half", [(4000, 100, True), (8191, 5, True), (8192, 20, False), (8192, 21, True),
                                      (24000, 10, False),
                                      (24000, 52, False), (24000, 53, True), (32767, 128, True), (32768, 128, False),
                                      (4000, 129, False)])
def test_draw_form_by_atoms_and_draws(record, n, p, half):
    """Few draws per atom leave most lanes of the half-wavefront form idle."""
    calls = record(f"create:n={n},box={(n / 100) ** (1 / 3):.4f},p={p}", "set", "build", "forces")
    names = [r.split()[1] for r in calls[3][2] if r.startswith("launch")]
    assert any("k_draw_batches_half" in k for k in names) == half
