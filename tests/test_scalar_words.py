"""Words of the solver's scalar block that one launch both reads and writes, found in the sources.

Every wave of a kernel reads the block with loads of its own, and workgroups begin at different times: a word that one workgroup
writes while others may still read it can have two values in one workgroup, whose waves then part ways between barriers.  A
kernel of several workgroups may therefore write what it reads only where every reader is known to be done: behind
arrive_is_last, or, with the reason given here, in calls that do not read the word."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_16340_amd", "csrc")

ONE_WORKGROUP = {"k_al_begin", "k_al_reopen", "k_al_turn", "k_reopen", "k_commit", "k_retest", "k_clear_bail", "k_admit", "k_check_start",
                 "k_resident", "k_small_step"}
READ_AND_WRITTEN = {
    # the choice is read from the block only in calls that do not record it there (no records of the direction kernel)
    "k_fused_ring": {"alpha_ub"},
    # ... and `fresh`, of the block's copy, by workgroup 0 alone
    "k_ot_sums": {"alpha_ub", "branch", "fresh"},
    # all behind the arrival
    "k_ot_update_entropy": {"count", "head", "status"},
    "k_ls_logistic": {"ls_ok"},
    # behind the arrival, or (ls_ok, spec_ok) where what was read is not used or is the value written; status: see below
    "k_update_logistic": {"count", "f", "head", "ls_ok", "spec_ok", "status"},
    # written in calls that do not look at it first (reopen)
    "k_eval_finish": {"status"},
}


def bodies(text, pattern):
    """(name, parameters, body) of the functions that `pattern` begins"""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)
    for at in re.finditer(pattern, text):
        head = re.compile(r"\b(\w+)\s*\(").search(text, at.end())
        while head.group(1) in ("__launch_bounds__", "__attribute__", "amdgpu_waves_per_eu"):
            head = re.compile(r"\b(\w+)\s*\(").search(text, head.end())
        begin = text.index("{", head.end())
        depth, end = 1, begin + 1
        while depth:
            depth += {"{": 1, "}": -1}.get(text[end], 0)
            end += 1
        yield head.group(1), text[head.start():begin], text[begin:end]


def kernels():
    for name in sorted(os.listdir(CSRC)):
        yield from bodies(open(os.path.join(CSRC, name)).read(), r"__global__")


def words(signature, body):
    names = set(re.findall(r"\bScal\s*\*\s*(?:__restrict__\s*)?(\w+)", signature)) - {"host_scal"} | {"a.scal"}
    read, written = set(), set()
    for n in names:
        for m in re.finditer(r"(?<![\w.])" + re.escape(n) + r"->(\w+)(?:\[[^\]]*\])?\s*(\+=|-=|=(?!=))?", body):
            (written if m.group(2) else read).add((n, m.group(1)))
    return read, written


def test_words_read_and_written_in_one_launch():
    found = {}
    for name, signature, body in kernels():
        read, written = words(signature, body)
        if name not in ONE_WORKGROUP and read & written:
            found.setdefault(name, set()).update(word for _, word in read & written)
    assert found == READ_AND_WRITTEN


def test_the_entropy_search_reads_nothing_that_it_writes():
    seen = {}
    for name, signature, body in kernels():
        if name.startswith("k_ot_ls_"):
            seen[name] = words(signature, body)
    read, written = seen["k_ot_ls_fine"]
    assert len(seen) == 3 and ("scal", "ls_ok") in written and ("scal", "status") in read
    for name, (read, written) in seen.items():
        assert not read & written, name


def test_a_workgroup_agrees_whether_the_solver_is_parked():
    """k_update_logistic parks the solver (status) without an arrival: only workgroup 0, which writes the word, may leave by what a
    wave has read of it, the others by the sum that all of their waves make together."""
    body = [b for name, _, b in kernels() if name == "k_update_logistic"][0]
    parks = body.index("scal->status = kStatusBail")
    assert body.count("kStatusBail") == 1 and body[:parks].rstrip().count("return;") == 1
    assert body[:parks].count("scal->status") == 1 and "const bool running = scal->status == LBFGSB_RUNNING;" in body[:parks]
    assert "if (!running && !(short_seq && blockIdx.x > 0)) return;" in body[:parks]
    assert "running ? 0.0 : NAN" in body[:parks] and "isfinite(df)" in body[:parks]


def test_a_run_that_is_over_is_not_opened_again():
    """The host goes on behind the last turn until it sees that the run is over: every way back to a running solver looks at the
    device's own word for that first."""
    by_name = {name: (signature, body) for name, signature, body in kernels()}
    assert by_name["k_al_reopen"][1].index("state->done) return;") < by_name["k_al_reopen"][1].index("scal->status = LBFGSB_RUNNING")
    signature, body = by_name["k_eval_finish"]
    first = body.index("return;")
    assert "over" in signature and "if (reopen ? over && *over :" in body[:first] and first < body.index("scal->status = LBFGSB_RUNNING")
    turn = next(b for n, _, b in bodies(open(os.path.join(CSRC, "api.hip")).read(), r"\nvoid (?=enqueue_turn)") if n == "enqueue_turn")
    assert "if (!own_test) hipLaunchKernelGGL(k_al_reopen" in turn and "enqueue_eval(s, 0, true, own_test, nullptr, &al->state->done)" in turn
    assert by_name["k_al_turn"][1].index("state->done) return;") < by_name["k_al_turn"][1].index("retest_point")


def test_algorithm_4_returns_from_an_idle_device():
    """lbfgsb_auglag_solve synchronises, a run that is refused on the way included: the steps behind its end still use the workspace, and
    what the device has written for the host is whole when it is idle."""
    solve = next(b for n, _, b in bodies(open(os.path.join(CSRC, "api.hip")).read(), r"\nint (?=lbfgsb_auglag_solve)") if n == "lbfgsb_auglag_solve")
    assert solve.count("end->nonfinite") == 1
    behind_the_loop = solve[solve.rindex("run.begin(0);"):]
    assert behind_the_loop.index("HIP_TRY(read_scal(s));") < behind_the_loop.index("end->nonfinite")
