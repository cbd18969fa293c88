"""Parity of the HIP program-counter virtual machine with its oracle, through the C ABI, on a real MI355X.
Everything is 64-bit integer work: outputs, step counts, active-member counts and the schedule trace are
compared bit for bit."""
import numpy as np
import pytest

from oracle import pcvm_ref as V
from paper_1910_11141_amd import pcvm_programs as PP

pytestmark = pytest.mark.gpu


def gpu(program, inputs, depth, **kw):  # kw: max_steps, trace_capacity, queued
    import torch
    from paper_1910_11141_amd import pcvm
    ins = torch.as_tensor(np.ascontiguousarray(np.asarray(inputs, dtype=np.int64).reshape(program.n_inputs, -1))).cuda()
    out, stats, trace = pcvm.pcvm_run(program, ins, depth, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy(), stats, None if trace is None else trace.cpu().numpy()


def inputs_for(name, batch, seed):
    rng = np.random.default_rng(seed)
    if name == "fibonacci":
        return rng.integers(0, 15, size=(1, batch))
    if name == "collatz_steps":
        return rng.integers(1, 5000, size=(1, batch))
    if name == "gcd":
        return rng.integers(0, 10**9, size=(2, batch))
    if name == "parity":
        return rng.integers(0, 60, size=(1, batch))
    if name == "binomial":
        n = rng.integers(0, 11, size=batch)
        return np.stack([n, (rng.random(batch) * (n + 1)).astype(np.int64)])
    m = rng.integers(0, 3, size=batch)
    return np.stack([m, rng.integers(0, 5, size=batch)])


def test_fibonacci_worked_example_outputs_and_schedule():
    """The batch of Figure 3: same outputs and the same sequence of (block, active members) as Algorithm 2."""
    P = PP.fibonacci()
    want, st, trace = V.run(P, [6, 7, 8, 9], 12)
    out, stats, tr = gpu(P, [6, 7, 8, 9], 12, trace_capacity=1000)
    assert list(out) == [13, 21, 34, 55] == list(want)
    assert stats["steps"] == st["steps"] == 458 and stats["active_member_steps"] == st["active_member_steps"]
    assert [tuple(r) for r in tr[: st["steps"]]] == trace
    assert (tr[st["steps"]:] == -1).all()


@pytest.mark.parametrize("batch", [1, 63, 64, 65, 257, 1000])
@pytest.mark.parametrize("name", sorted(PP.ALL))
def test_programs_match_the_oracle_on_ragged_batches(name, batch):
    P = PP.ALL[name]()
    ins = inputs_for(name, batch, seed=batch)
    want, st, trace = V.run(P, ins, 80, group=64)
    out, stats, tr = gpu(P, ins, 80, trace_capacity=len(trace))
    assert np.array_equal(out, want)
    assert stats["steps"] == st["steps"] and stats["active_member_steps"] == st["active_member_steps"]
    assert stats["issued_member_steps"] == st["issued_member_steps"] and stats["n_groups"] == (batch + 63) // 64
    assert [tuple(r) for r in tr] == trace            # group 0 took the same blocks in the same order


def test_large_batch_against_the_closed_form_and_sampled_members():
    P = PP.fibonacci()
    rng = np.random.default_rng(5)
    ns = rng.integers(0, 21, size=200_000)
    out, stats, _ = gpu(P, ns, 32)
    fib = np.ones(22, dtype=np.int64)
    for i in range(2, 22):
        fib[i] = fib[i - 1] + fib[i - 2]
    assert np.array_equal(out, fib[ns])
    pick = rng.choice(ns.size, 64, replace=False)
    assert np.array_equal(out[pick], V.run(P, ns[pick], 32)[0])
    assert 0.0 < stats["utilization"] <= 1.0
    again, stats2, _ = gpu(P, ns, 32)
    assert np.array_equal(again, out) and stats2["steps"] == stats["steps"]


def test_equal_inputs_keep_every_lane_busy():
    out, stats, _ = gpu(PP.fibonacci(), [11] * 128, 16)
    assert (out == 144).all() and stats["utilization"] == 1.0


def test_limits_are_reported_not_trapped():
    from paper_1910_11141_amd import pcvm
    P = PP.fibonacci()
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(P, [3, 12, 2, 1], 6)
    assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(PP.parity(), [100] * 70, 50)
    assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(P, [15], 20, max_steps=100)
    assert e.value.code == pcvm.PCVM_E_STEP_LIMIT
    bad = PP.fibonacci()
    bad.ops["kind"][1] = PP.POP             # pops `ret`, which is never pushed
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(bad, [0, 5], 8)
    assert e.value.code == pcvm.PCVM_E_STACK_UNDERFLOW
    out, _, _ = gpu(P, [3, 4], 6)           # the library is still usable afterwards
    assert list(out) == [3, 5]


def test_maximum_stack_depth_and_variable_count():
    from paper_1910_11141_amd import pcvm
    P = PP.parity()
    ns = np.array([4094, 4095, 17, 0] * 20)       # 4095 nested calls need 4096 program-counter entries
    out, stats, _ = gpu(P, ns, pcvm.PCVM_MAX_DEPTH)
    assert list(out) == [1 - int(n) % 2 for n in ns]
    want, st, _ = V.run(P, ns[:8], pcvm.PCVM_MAX_DEPTH)
    assert np.array_equal(out[:8], want)
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(P, [4096], pcvm.PCVM_MAX_DEPTH)
    assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
    # a program that uses all 16 variables: a chain of copies and additions through every one of them
    b = PP._Builder("wide", [f"v{i}" for i in range(16)], 1, "v15")
    ops = [PP.update(f"v{i}", PP.ADDI, f"v{i - 1}", imm=i) for i in range(1, 16)]
    b.block("only", 1, ops, (PP.RETURN,))
    wide = b.build()
    xs = np.arange(100)
    out, _, _ = gpu(wide, xs, 4)
    assert np.array_equal(out, xs + sum(range(1, 16)))
    assert np.array_equal(V.run(wide, xs, 4)[0], out)


# ------------------------------------------------------------------ members handed out from a queue

@pytest.mark.parametrize("batch", [1, 65, 1000, 70_000])
@pytest.mark.parametrize("name", sorted(PP.ALL))
def test_queued_runs_give_the_same_outputs(name, batch):
    P = PP.ALL[name]()
    ins = inputs_for(name, batch, seed=batch + 1)
    static, st_static, _ = gpu(P, ins, 80)
    queued, st_queued, _ = gpu(P, ins, 80, queued=True, policy=batch % 2)
    assert np.array_equal(queued, static)
    assert st_queued["active_member_steps"] == st_static["active_member_steps"]    # the same blocks per member
    if batch <= 1000:
        assert np.array_equal(static, V.run(P, ins, 80)[0])


def test_queue_keeps_lanes_busy_on_unequal_work():
    P = PP.fibonacci()
    ns = np.random.default_rng(9).integers(1, 21, size=1 << 20)
    static, st_static, _ = gpu(P, ns, 32)
    queued, st_queued, _ = gpu(P, ns, 32, queued=True)
    fuller, st_fuller, _ = gpu(P, ns, 32, queued=True, policy=1)
    assert np.array_equal(static, queued) and np.array_equal(static, fuller)
    assert st_static["utilization"] < st_queued["utilization"] < st_fuller["utilization"]
    assert st_fuller["active_member_steps"] == st_static["active_member_steps"]
    assert st_queued["n_groups"] < st_static["n_groups"]
    print("utilization static / queued / queued most-waiting:", st_static["utilization"], st_queued["utilization"],
          st_fuller["utilization"], "ms", st_static["kernel_ms"], st_queued["kernel_ms"], st_fuller["kernel_ms"])


def test_queued_limits_are_reported_and_other_members_finish():
    from paper_1910_11141_amd import pcvm
    P = PP.fibonacci()
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(P, [3, 12, 2, 1] * 50, 6, queued=True)
    assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
    with pytest.raises(pcvm.PcvmError) as e:
        gpu(P, [15] * 300, 20, max_steps=100, queued=True)
    assert e.value.code == pcvm.PCVM_E_STEP_LIMIT
    out, _, _ = gpu(P, [3, 4] * 100, 6, queued=True)
    assert list(out) == [3, 5] * 100


# ------------------------------------------------------------------ programs on either side of 64 operations and blocks

def long_program(n_ops, n_blocks):
    """n_blocks blocks that share n_ops operations: every function, pushes and pops of two variables, a loop over n."""
    b = PP._Builder("long", ["n", "x", "y", "c", "s"], 1, "s")
    body = [PP.update("x", PP.ADDI, "n", imm=7), PP.update("s", PP.ADD, "s", "x"), PP.push("y", PP.MUL, "x", "n"), PP.update("y", PP.SUB, "y", "x"),
            PP.push("x", PP.MOD, "y", "x"), PP.update("c", PP.LT, "x", "y"), PP.update("x", PP.ADD, "x", "c"),
            PP.update("c", PP.COPY, "x"), PP.pop("x"), PP.update("x", PP.ANDI, "x", imm=(1 << 40) - 1), PP.update("y", PP.MULI, "y", imm=-3),
            PP.update("c", PP.SHRI, "y", imm=3), PP.update("x", PP.ADD, "x", "c"), PP.pop("y"), PP.update("s", PP.ADD, "s", "c"), PP.update("c", PP.LE, "x", "y"),
            PP.update("c", PP.EQ, "c", "n"), PP.update("y", PP.CONST, imm=-(1 << 35)), PP.update("s", PP.MULI, "s", imm=31), PP.update("s", PP.SUB, "s", "y")]
    ops = [body[i % len(body)] for i in range(n_ops - 2)]
    per = [ops[i * len(ops) // (n_blocks - 2):(i + 1) * len(ops) // (n_blocks - 2)] for i in range(n_blocks - 2)]
    for i, o in enumerate(per):
        b.block(f"b{i}", i, o, (PP.JUMP, f"b{i + 1}" if i + 1 < len(per) else "test"))
    b.block("test", 98, [PP.update("n", PP.ADDI, "n", imm=-1), PP.update("c", PP.LEI, "n", imm=0)], (PP.BRANCH, "c", "done", "b0"))
    b.block("done", 99, [], (PP.RETURN,))
    return b.build()


@pytest.mark.parametrize("n_ops,n_blocks", [(18, 3), (64, 9), (65, 9), (50, 64), (50, 65), (130, 70)])
def test_small_and_general_interpreters_match_the_oracle(n_ops, n_blocks):
    P = long_program(n_ops, n_blocks)
    assert len(P.ops) == n_ops and len(P.blocks) == n_blocks
    ins = np.random.default_rng(n_ops).integers(1, 9, size=150)
    want, st, trace = V.run(P, ins, 40, group=64)
    out, stats, tr = gpu(P, ins, 40, trace_capacity=len(trace))
    assert np.array_equal(out, want) and stats["steps"] == st["steps"]
    assert [tuple(r) for r in tr] == trace
    for policy in (0, 1):
        assert np.array_equal(gpu(P, ins, 40, queued=True, policy=policy)[0], want)


@pytest.mark.parametrize("depth", [1, 2, 3, 17, 64, 300])
def test_stack_rings_spill_and_refill_at_any_depth(depth):
    """Deep recursion through two pushed arguments: every ring length, entries that leave the ring and come back."""
    P = PP.ackermann()
    from paper_1910_11141_amd import pcvm
    ins = np.array([[0, 1, 2, 2, 3] * 30, [3, 4, 3, 0, 3] * 30])
    try:
        want = V.run(P, ins, depth)[0]
    except Exception:
        with pytest.raises(pcvm.PcvmError) as e:
            gpu(P, ins, depth)
        assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
        with pytest.raises(pcvm.PcvmError):
            gpu(P, ins, depth, queued=True, policy=1)
        return
    for kw in (dict(), dict(queued=True), dict(queued=True, policy=1)):
        assert np.array_equal(gpu(P, ins, depth, **kw)[0], want)


def test_queued_batches_around_the_number_of_lanes_that_take_members():
    """The first member of a lane is handed out without the queue: batches of one member, of as many as there are lanes, of
    one more and one less, at each of the group shapes."""
    import torch
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(9)
    P = PP.gcd()
    for batch in (1, 2, 63, 64, 65, simds - 1, simds, simds + 1, 2 * simds, 7 * simds - 3, 64 * simds, 64 * simds + 1, 192 * simds - 1,
                  192 * simds, 192 * simds + 1, 192 * simds + 4099):
        ins = rng.integers(1, 10 ** 6, size=(2, batch))
        want = np.gcd(ins[0], ins[1])
        for policy in (0, 1):
            out, stats, _ = gpu(P, ins, 40, queued=True, policy=policy)
            assert np.array_equal(out, want), (batch, policy)


def call_program(n_pad, n_deep):
    """A recursion that pushes the value of every function and calls from joined blocks; n_pad blocks that only jump
    lengthen the chains and the table, and n_deep is how much deeper a call goes for each unit of its argument."""
    b = PP._Builder("calls", ["n", "x", "y", "c", "s", "t"], 1, "s")
    b.block("f", 1, [PP.update("c", PP.LEI, "n", imm=0)], (PP.BRANCH, "c", "base", "go"))
    b.block("base", 2, [PP.update("s", PP.ADDI, "s", imm=1), PP.pop("n")], (PP.RETURN,))
    pushes = [PP.push("x", PP.MUL, "n", "s"), PP.push("y", PP.MULI, "n", imm=-7), PP.push("t", PP.MOD, "x", "y"), PP.push("x", PP.SUB, "x", "t"),
              PP.push("y", PP.LT, "x", "y"), PP.push("t", PP.SHRI, "x", imm=2), PP.push("x", PP.EQI, "n", imm=2), PP.push("y", PP.LE, "t", "n")]
    pops = [PP.update("s", PP.ADD, "s", v) for v in ("x", "y", "t")] + [PP.pop(v) for v in ("y", "x", "t", "y", "x", "t", "y", "x")]
    b.block("go", 3, pushes, (PP.JUMP, "pad0" if n_pad else "call"))
    for i in range(n_pad):
        b.block(f"pad{i}", 10 + i, [], (PP.JUMP, f"pad{i + 1}" if i + 1 < n_pad else "call"))
    b.block("call", 4, [PP.push("n", PP.ADDI, "n", imm=-1)], (PP.PUSHJUMP, "f", "back"))
    b.block("back", 5, pops + [PP.update("c", PP.ANDI, "n", imm=n_deep)], (PP.BRANCH, "c", "again", "leave"))
    b.block("again", 6, [PP.update("n", PP.ADDI, "n", imm=-2)], (PP.PUSHJUMP, "f", "out"))
    b.block("leave", 7, [PP.pop("n")], (PP.RETURN,))
    b.block("out", 8, [], (PP.RETURN,))
    return b.build()


@pytest.mark.parametrize("n_pad,n_deep,top", [(0, 0, 40), (0, 3, 12), (23, 3, 12), (30, 1, 12), (31, 1, 12), (55, 0, 40)])
def test_calls_and_pushed_values_match_the_oracle(n_pad, n_deep, top):
    """Return addresses of 4 to 6 bits in 16 to 10 places of a register pair, spilled and read back; tables of entries in one
    set of registers and in two (from 39 blocks on); records that join up to four blocks, with and without a call."""
    P = call_program(n_pad, n_deep)
    ins = np.random.default_rng(n_pad).integers(0, top, size=130)
    for depth in (top // 2, 2 * top + 8, 4 * top + 40):
        try:
            want, st, trace = V.run(P, ins, depth, group=64)
        except V.StackOverflow:
            from paper_1910_11141_amd import pcvm
            for kw in (dict(), dict(queued=True), dict(queued=True, policy=1)):
                with pytest.raises(pcvm.PcvmError) as e:
                    gpu(P, ins, depth, **kw)
                assert e.value.code == pcvm.PCVM_E_STACK_OVERFLOW
            continue
        out, stats, tr = gpu(P, ins, depth, trace_capacity=len(trace))
        assert np.array_equal(out, want) and stats["steps"] == st["steps"]
        assert [tuple(r) for r in tr] == trace
        for policy in (0, 1):
            out, stats, _ = gpu(P, ins, depth, queued=True, policy=policy)
            assert np.array_equal(out, want) and stats["active_member_steps"] == st["active_member_steps"]


def test_remainders_of_small_large_and_negative_numbers():
    """Numbers below 2^32 (a reciprocal in binary64) and all others, in one wave and apart, at the edges of a quotient."""
    P = PP.gcd()
    rng = np.random.default_rng(3)
    small = np.array([0, 1, 2, 3, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 2 ** 32 - 2, 2 ** 32 - 1])
    b = np.concatenate([rng.integers(1, 2 ** 32, 2000), rng.integers(1, 2 ** 16, 2000)])
    edges = np.minimum(b * rng.integers(1, 2 ** 16, b.size) + rng.integers(-1, 2, b.size), 2 ** 32 - 1)
    wide = np.array([-1, -2, 2 ** 32, 2 ** 33 + 5, -2 ** 63, 2 ** 63 - 1, 2 ** 53 + 1, -7])
    for x, y in ((np.repeat(small, small.size), np.tile(small, small.size)), (edges, b), (np.maximum(edges, 0), rng.permutation(b)),
                 (np.repeat(wide, wide.size), np.tile(wide, wide.size)), (rng.permutation(np.tile(small, 8)), rng.permutation(np.tile(wide, 9)))):
        ins = np.stack([x, y])
        want = V.run(P, ins, 120)[0]
        for kw in (dict(), dict(queued=True, policy=1)):
            assert np.array_equal(gpu(P, ins, 120, **kw)[0], want)
