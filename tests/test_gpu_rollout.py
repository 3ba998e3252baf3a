"""GPU parity of tp_rollout (fused actor + sampling + env step + trajectory
store) against a teacher-forced oracle replay, at sizes the oracle finishes
in seconds: several workgroups of envs, ragged tails, every actor shape
family (bf16 256- to 1024-wide on the role-split kernel, fp32 and other bf16
shapes on the four-env kernel, the rest on the generic kernel, multi-agent), plus
determinism, split/resume, and envs whose start row leaves no room."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_common import (bits16, build_problem, compare_rollout, oracle_replay,
                        rel_check, say)
from paper_2111_05188_amd import tp

pytestmark = pytest.mark.gpu

SEED = 0x5EED0FF12C


def _run_case(cfg, E, L, rows=None, n_agents=1, cmp_ids=None, step0=0):
    rows = cfg.T1 if rows is None else rows
    c = cfg.with_(N=rows - 1, E=E, n_agents=n_agents)
    mk = W.make_market(c)
    t0 = W.make_t0(c)
    pb, params = build_problem(c, mk, t0)
    pb.reset()
    say(f"[rollout] {cfg.name} E={E} L={L} agents={n_agents} rows={rows}")
    pb.rollout(SEED, step0, L)
    torch.cuda.synchronize()
    ids = np.arange(E) if cmp_ids is None else np.asarray(cmp_ids)
    teacher = pb.traj.action[:L].index_select(
        1, torch.as_tensor(ids, device="cuda")).cpu().numpy()
    out = oracle_replay(c, mk, params, t0[ids], ids, SEED, L, teacher,
                        c.envs_per_agent, step0=step0)
    compare_rollout(c, pb, out, ids, L)
    cash, sh, t = out["final"]
    ids_t = torch.as_tensor(ids, device="cuda")
    assert np.array_equal(pb.state.cash.index_select(0, ids_t).cpu().numpy(), cash)
    assert np.array_equal(pb.state.shares.index_select(0, ids_t).cpu().numpy(), sh)
    assert np.array_equal(pb.state.t.index_select(0, ids_t).cpu().numpy(), t)
    ol = pb.traj.obs_last.index_select(0, ids_t)[:, :c.K_pad]
    g = bits16(ol) if c.dtype == "bf16" else ol.cpu().numpy()
    assert np.array_equal(g, out["obs_last"])
    return pb


def test_tiny_full():
    _run_case(W.get_config("tiny"), 64, 256)


def test_tiny_ragged_env_count():
    _run_case(W.get_config("tiny"), 7, 50)


def test_nasdaq_shape_small_market_ragged():
    # full n, I and 1001-512-512-100 bf16 actor; 3 workgroups, ragged tail
    _run_case(W.get_config("nasdaq100"), 37, 60, rows=40 * 390 + 1)


def test_ensemble_shape_three_agents_ragged():
    _run_case(W.get_config("ensemble"), 60, 40, rows=20 * 390 + 1, n_agents=3)


@pytest.mark.parametrize("L", [1, 2, 4, 5])
def test_nasdaq_shape_short_rollouts(L):
    """Rollouts shorter than, or not a multiple of, the role-split kernel's
    market batch of three steps: the partial final batch, the bootstrap
    observation row and the final state."""
    _run_case(W.get_config("nasdaq100"), 20, L, rows=6 * 390 + 1)


def test_stress_shape_small():
    _run_case(W.get_config("stress"), 20, 30, rows=20 * 390 + 1)


@pytest.mark.parametrize("I,H,L", [(4, 512, 50), (4, 256, 4), (4, 768, 5), (4, 1024, 3),
                                   (10, 512, 50), (10, 256, 4), (10, 768, 5), (10, 1024, 3)])
def test_role_split_other_markets(I, H, L):
    """The role-split kernel on the 100-stock markets with 4 and 10
    indicators per stock (601 and 1201 inputs: 20 and 40 k-steps, observation
    rows of 608 and 1,216 columns), at every width, three workgroups with a
    ragged tail, rollouts that end inside a market batch."""
    cfg = W.get_config("nasdaq100").with_(n_ind=I, hidden=(H, H))
    pb = _run_case(cfg, 37, L, rows=20 * 390 + 1)
    assert tp.rollout_path(pb.mkt, pb.actor) == 1


@pytest.mark.parametrize("I,H,agents,E", [(10, 768, 3, 60), (4, 512, 2, 34), (10, 512, 1, 1),
                                          (10, 1024, 1, 17)])
def test_role_split_agents_and_env_counts(I, H, agents, E):
    """Several agents per launch (each agent's blocks in its own run of
    workgroups, ragged per agent), a single env, and one env past a
    workgroup, on the market-batch and single-step paths."""
    cfg = W.get_config("nasdaq100").with_(n_ind=I, hidden=(H, H))
    pb = _run_case(cfg, E, 20, rows=20 * 390 + 1, n_agents=agents)
    assert tp.rollout_path(pb.mkt, pb.actor) == 1


@pytest.mark.parametrize("H,L", [(256, 50), (256, 4), (768, 50), (768, 3)])
def test_role_split_other_widths(H, L):
    """The role-split kernel at its other hidden widths (256: market batches
    of three steps; 768: of two), three workgroups with a ragged tail, and
    rollouts that end inside a batch."""
    pb = _run_case(W.get_config("nasdaq100").with_(hidden=(H, H)), 37, L, rows=20 * 390 + 1)
    assert tp.rollout_path(pb.mkt, pb.actor) == 1


def test_dow_shape_small():
    _run_case(W.get_config("dow30"), 9, 300, rows=2521)


def test_bf16_actor_of_another_shape():
    # a bf16 actor outside the role-split kernel's shapes (301 inputs, 256-wide
    # layers) runs the four-env kernel
    _run_case(W.get_config("dow30").with_(dtype="bf16"), 21, 120, rows=2521)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_largest_market(dtype):
    # 128 stocks x 8 indicators (n * n_ind = 1024, the largest market the
    # boundary takes; 1281 inputs) on the four-env kernel, fp32 and bf16
    cfg = W.get_config("tiny").with_(n=128, n_ind=8, dtype=dtype, hidden=(128, 128))
    pb = _run_case(cfg, 20, 40)
    assert tp.rollout_path(pb.mkt, pb.actor) == 0


GENERIC, FOUR = 0, 2   # tp_rollout_kernel


@pytest.mark.parametrize("n,I,hidden,E,L,agents,dtype,kernel", [
    (1, 0, (4, 4), 1, 1, 1, "f32", FOUR),          # one stock, no indicators, one k-block
    (8, 8, (16, 16), 5, 2, 1, "f32", FOUR),        # holdings end on a k-block's edge
    (5, 4, (96, 36), 1030, 3, 1, "f32", FOUR),     # eight envs a workgroup, a ragged last one
    (33, 8, (320, 192), 9, 4, 3, "f32", FOUR),     # eight stocks a lane, two tile groups of layer 1
    (20, 8, (1024, 500), 6, 3, 1, "f32", FOUR),    # four groups; layers that stream
    (5, 4, (1028, 64), 6, 3, 1, "f32", GENERIC),   # wider than the kernel
    (31, 3, (256, 128), 1100, 3, 2, "bf16", FOUR),
    (64, 4, (128, 384), 21, 2, 3, "bf16", FOUR),
    (128, 8, (640, 128), 7, 3, 1, "bf16", GENERIC),
    (100, 5, (256, 384), 2064, 2, 1, "bf16", FOUR),    # sixteen envs a workgroup
])
def test_four_env_kernel_edges(n, I, hidden, E, L, agents, dtype, kernel):
    cfg = W.get_config("tiny").with_(name=f"four-{n}", n=n, n_ind=I, hidden=hidden, dtype=dtype)
    ids = None if E < 100 else np.r_[0:5, E // agents - 3:E // agents + 3, E - 9:E]
    ids = ids if ids is None else np.unique(ids[ids < E])
    pb = _run_case(cfg, E, L, rows=8, n_agents=agents, cmp_ids=ids)
    assert tp.rollout_path(pb.mkt, pb.actor) == 0
    assert tp.rollout_kernel(pb.mkt, pb.actor) == kernel


# Every instantiation of the four-env kernel: tile groups (GT, TW) by the
# hidden widths, two or eight stocks a lane, and envs a workgroup by the env
# count (4 up to 256 workgroups, then 8, for bf16 then 16).  The env counts
# end inside a workgroup's second group of four; several agents are ragged each.
@pytest.mark.parametrize("n,I", [(5, 4), (33, 3)])
@pytest.mark.parametrize("hidden,dtype", [
    ((64, 32), "f32"), ((128, 128), "f32"), ((320, 192), "f32"), ((256, 256), "f32"),
    ((1024, 64), "f32"),
    ((128, 128), "bf16"), ((384, 384), "bf16"), ((256, 256), "bf16"), ((128, 768), "bf16"),
])
@pytest.mark.parametrize("E,agents", [(11, 1), (1037, 1), (3 * 345, 3), (2063, 1), (3 * 691, 3)])
def test_four_env_kernel_variants(n, I, hidden, dtype, E, agents):
    cfg = W.get_config("tiny").with_(name=f"four-{n}", n=n, n_ind=I, hidden=hidden, dtype=dtype)
    epa = E // agents
    ids = np.unique(np.r_[0:min(9, epa), epa - 3:epa, E - 5:E])
    pb = _run_case(cfg, E, 3, rows=8, n_agents=agents, cmp_ids=ids)
    assert tp.rollout_kernel(pb.mkt, pb.actor) == FOUR


@pytest.mark.parametrize("n,I,hidden,dtype,kernel", [
    (5, 4, (64, 64), "f32", FOUR), (33, 3, (320, 192), "f32", FOUR), (30, 8, (256, 256), "f32", FOUR),
    (5, 4, (1028, 64), "f32", GENERIC),
    (30, 8, (256, 256), "bf16", FOUR), (33, 3, (384, 384), "bf16", FOUR),
    (100, 8, (384, 256), "bf16", FOUR), (100, 8, (512, 384), "bf16", GENERIC),
])
def test_results_do_not_depend_on_the_number_of_envs(n, I, hidden, dtype, kernel):
    """The first envs of a call alone give the same bits as among 1,040 and
    2,064 envs, where workgroups take more envs each (and a bf16 kernel chosen
    by the number of envs would be another one)."""
    cfg = W.get_config("tiny").with_(name=f"envs-{n}", n=n, n_ind=I, hidden=hidden, dtype=dtype,
                                     N=30, L=6)
    mk = W.make_market(cfg)
    runs = []
    for E in (11, 1040, 2064):
        t0 = np.arange(E, dtype=np.int64) % 20
        pb, _ = build_problem(cfg.with_(E=E), mk, t0)
        pb.reset()
        say(f"[rollout] {E} envs, {n} stocks {hidden} {dtype}")
        pb.rollout(SEED, 0, 6)
        torch.cuda.synchronize()
        assert tp.rollout_kernel(pb.mkt, pb.actor) == kernel
        runs.append(pb)
    for pb in runs[1:]:
        for name in ("action", "logp", "reward", "mu_tap", "cash_tap", "shares_tap", "obs"):
            a, b = getattr(runs[0].traj, name), getattr(pb.traj, name)
            assert torch.equal(a[:, :11], b[:, :11]), name
        assert torch.equal(runs[0].traj.obs_last, pb.traj.obs_last[:11])


def test_bf16_100_stock_actor_outside_the_role_split_shapes():
    # unequal hidden widths (512-256) on the 100 x 8 market: the generic kernel
    # takes it, with the same results contract
    cfg = W.get_config("nasdaq100").with_(hidden=(512, 256))
    pb = _run_case(cfg, 21, 30, rows=20 * 390 + 1)
    assert tp.rollout_path(pb.mkt, pb.actor) == 0


def test_deterministic_and_resumable():
    """Two identical runs are bitwise equal; rollout(L) equals rollout(j)
    followed by rollout(L-j, step0=j) from the saved state."""
    cfg = W.get_config("nasdaq100").with_(N=20 * 390, E=40)
    mk = W.make_market(cfg)
    t0 = W.make_t0(cfg)
    L, j = 40, 15
    runs = []
    for _ in range(2):
        pb, _ = build_problem(cfg, mk, t0)
        pb.reset()
        say("[rollout] determinism run")
        pb.rollout(SEED, 0, L)
        torch.cuda.synchronize()
        runs.append(pb)
    a, b = runs
    # only the first L rows were written (the store holds a full episode)
    for name in ("action", "logp", "reward", "done", "cash_tap", "shares_tap", "obs"):
        assert torch.equal(getattr(a.traj, name)[:L], getattr(b.traj, name)[:L]), name
    # split run
    pb, _ = build_problem(cfg, mk, t0)
    pb.reset()
    t1 = tp.TrajT.alloc(j, cfg.E, cfg.n, cfg.K_pad, torch.bfloat16, taps=True, obs_last=True)
    t2 = tp.TrajT.alloc(L - j, cfg.E, cfg.n, cfg.K_pad, torch.bfloat16, taps=True, obs_last=True)
    say("[rollout] split run")
    pb.rollout(SEED, 0, j, traj=t1)
    pb.rollout(SEED, j, L - j, traj=t2)
    torch.cuda.synchronize()
    for name in ("action", "logp", "reward", "done", "cash_tap", "shares_tap", "obs"):
        full = getattr(a.traj, name)[:L]
        assert torch.equal(full[:j], getattr(t1, name)), name
        assert torch.equal(full[j:], getattr(t2, name)), name
    assert torch.equal(t1.obs_last, a.traj.obs[j])
    assert torch.equal(t2.obs_last, a.traj.obs_last)
    for s in ("cash", "shares", "t"):
        assert torch.equal(getattr(pb.state, s), getattr(a.state, s)), s


@pytest.mark.parametrize("n,I,hidden,dtype,E", [
    (5, 4, (64, 64), "f32", 11), (33, 3, (256, 128), "f32", 1037),
    (30, 8, (256, 256), "bf16", 1100), (33, 3, (384, 384), "bf16", 2063),
])
def test_four_env_kernel_resumes(n, I, hidden, dtype, E):
    """rollout(9) equals rollout(4) and rollout(5, step0=4) from the saved state,
    with 4, 8 and 16 envs a workgroup (an odd split: both row buffers start)."""
    cfg = W.get_config("tiny").with_(name=f"resume-{n}", n=n, n_ind=I, hidden=hidden, dtype=dtype,
                                     N=30, E=E, L=9)
    mk = W.make_market(cfg)
    t0 = np.arange(E, dtype=np.int64) % 20
    whole, _ = build_problem(cfg, mk, t0)
    split, _ = build_problem(cfg, mk, t0)
    assert tp.rollout_kernel(whole.mkt, whole.actor) == FOUR
    whole.reset()
    split.reset()
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    parts = [tp.TrajT.alloc(k, E, n, cfg.K_pad, dt, taps=True, obs_last=True) for k in (4, 5)]
    say(f"[rollout] resume, {n} stocks {hidden} {dtype}, {E} envs")
    whole.rollout(SEED, 0, 9)
    split.rollout(SEED, 0, 4, traj=parts[0])
    split.rollout(SEED, 4, 5, traj=parts[1])
    torch.cuda.synchronize()
    for name in ("action", "logp", "reward", "done", "cash_tap", "shares_tap", "mu_tap", "obs"):
        both = torch.cat([getattr(q, name) for q in parts])
        assert torch.equal(getattr(whole.traj, name)[:9], both), name
    assert torch.equal(parts[0].obs_last, whole.traj.obs[4])
    assert torch.equal(parts[1].obs_last, whole.traj.obs_last)
    for name in ("cash", "shares", "t"):
        assert torch.equal(getattr(whole.state, name), getattr(split.state, name)), name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_agents_of_one_call_equal_single_calls(dtype):
    """Three agents of 700 envs in one call: every agent's means on the first
    bar are those of a call over it alone (8 or 16 envs a workgroup against 4
    or 8; the action noise is drawn per agent, so only the means compare)."""
    cfg = W.get_config("tiny").with_(name="agents", n=30, n_ind=8, hidden=(256, 128), dtype=dtype,
                                     N=30, E=2100, n_agents=3, L=1)
    mk = W.make_market(cfg)
    t0 = np.arange(2100, dtype=np.int64) % 20
    pb, (Wl, b, ls) = build_problem(cfg, mk, t0)
    assert tp.rollout_kernel(pb.mkt, pb.actor) == FOUR
    pb.reset()
    pb.rollout(SEED, 0, 1)
    for a in range(3):
        sl = slice(a, a + 1)
        one, _ = build_problem(cfg.with_(E=700, n_agents=1), mk, t0[700 * a:700 * (a + 1)],
                               params=([w[sl] for w in Wl], [x[sl] for x in b], ls[sl]))
        one.reset()
        say(f"[rollout] agent {a} alone, {dtype}")
        one.rollout(SEED, 0, 1)
        torch.cuda.synchronize()
        assert torch.equal(pb.traj.mu_tap[0, 700 * a:700 * (a + 1)], one.traj.mu_tap[0]), a


def test_env_without_room_is_not_stepped():
    cfg = W.get_config("tiny")
    mk = W.make_market(cfg)
    t0 = np.zeros(20, np.int64)
    pb, _ = build_problem(cfg.with_(E=20), mk, t0, E=20, envs_per_agent=20)
    pb.state = tp.StateT.empty(20, cfg.n, count_invalid=True)
    pb.reset()
    assert pb.state.n_invalid.item() == 0
    # env 3 starts too late for L steps; env 4 has an invalid (negative) row
    pb.state.t[3] = cfg.T1 - 10
    pb.state.t[4] = -1
    say("[rollout] envs without room")
    pb.rollout(SEED, 0, 50)
    torch.cuda.synchronize()
    r = pb.traj.reward[:50].cpu().numpy()
    assert np.isnan(r[:, 3]).all() and np.isnan(r[:, 4]).all()
    assert np.isfinite(r[:, [0, 1, 2, 5]]).all()
    assert (pb.traj.done[:50].cpu().numpy()[:, 3] == 0).all()
    assert np.isnan(pb.traj.action[:50, 3].cpu().numpy()).all()
    assert np.isnan(pb.traj.mu_tap[:50, [3, 4]].cpu().numpy()).all()
    assert np.isfinite(pb.traj.mu_tap[:50, [0, 1, 2, 5]].cpu().numpy()).all()
    assert pb.state.t[3].item() == cfg.T1 - 10 and pb.state.t[4].item() == -1
    assert pb.state.t[0].item() == 50
    assert pb.state.n_invalid.item() == 2
    # the host check names the first env without room
    with pytest.raises(tp.TPError) as ei:
        tp.check_starts(pb.state.t.cpu().numpy(), cfg.T1, 50)
    assert ei.value.code == tp.TP_ERANGE and "env 3" in str(ei.value)


def test_env_without_room_role_split_kernel():
    """The same on the role-split kernel (100-stock bf16 actor): an env
    whose start row leaves no room is counted, its rows are NaN, and the
    envs sharing its waves are stepped as usual."""
    cfg = W.get_config("nasdaq100").with_(N=4 * 390, E=20)
    mk = W.make_market(cfg)
    t0 = W.make_t0(cfg)
    pb, params = build_problem(cfg, mk, t0)
    assert tp.rollout_path(pb.mkt, pb.actor) == 1
    pb.state = tp.StateT.empty(20, cfg.n, count_invalid=True)
    pb.reset()
    pb.state.t[6] = cfg.T1 - 5
    pb.state.t[9] = -7
    say("[rollout] role-split kernel, envs without room")
    pb.rollout(SEED, 0, 30)
    torch.cuda.synchronize()
    assert pb.state.n_invalid.item() == 2
    r = pb.traj.reward[:30].cpu().numpy()
    assert np.isnan(r[:, [6, 9]]).all() and np.isfinite(np.delete(r, [6, 9], axis=1)).all()
    assert np.isnan(pb.traj.mu_tap[:30, [6, 9]].cpu().numpy()).all()
    ids = np.array([0, 7, 8, 19])
    teacher = pb.traj.action[:30].index_select(1, torch.as_tensor(ids, device="cuda")).cpu().numpy()
    out = oracle_replay(cfg, mk, params, t0[ids], ids, SEED, 30, teacher, cfg.envs_per_agent)
    compare_rollout(cfg, pb, out, ids, 30)


@pytest.mark.parametrize("n,I,hidden,dtype,E,kernel", [
    (5, 4, (1028, 64), "f32", 21, GENERIC),
    (5, 4, (512, 128), "bf16", 37, GENERIC),
    (5, 4, (64, 64), "f32", 1037, FOUR),
    (33, 3, (256, 128), "bf16", 2063, FOUR),
])
def test_env_without_room_other_kernels(n, I, hidden, dtype, E, kernel):
    """Envs that cannot be stepped on the generic kernel and on the four-env
    kernel with 8 and 16 envs a workgroup: NaN rows, done 0, taps that repeat
    the state, the state unchanged, both counted; the others as the oracle."""
    cfg = W.get_config("tiny").with_(name=f"room-{n}", n=n, n_ind=I, hidden=hidden, dtype=dtype,
                                     N=40, E=E, L=20)
    mk = W.make_market(cfg)
    t0 = W.make_t0(cfg)
    pb, params = build_problem(cfg, mk, t0)
    assert tp.rollout_kernel(pb.mkt, pb.actor) == kernel
    pb.state = tp.StateT.empty(E, n, count_invalid=True)
    pb.reset()
    bad = [6, E - 2]
    pb.state.t[bad[0]], pb.state.t[bad[1]] = cfg.T1 - 5, -7
    pb.state.cash[bad[0]] = 1234.5
    pb.state.shares[bad[0], n - 1] = 3
    say(f"[rollout] envs without room, {n} stocks {hidden} {dtype}, {E} envs")
    pb.rollout(SEED, 0, 20)
    torch.cuda.synchronize()
    tr = pb.traj
    assert pb.state.n_invalid.item() == 2
    for x in (tr.action, tr.logp, tr.reward, tr.mu_tap, tr.asset_tap):
        assert torch.isnan(x[:20, bad]).all()
    assert (tr.done[:20, bad] == 0).all()
    assert (tr.cash_tap[:20, bad[0]] == 1234.5).all()
    want = torch.zeros(n, dtype=torch.int32, device="cuda")
    want[n - 1] = 3
    assert (tr.shares_tap[:20, bad[0]] == want).all() and (tr.shares_tap[:20, bad[1]] == 0).all()
    assert pb.state.t[bad].tolist() == [cfg.T1 - 5, -7]
    assert pb.state.cash[bad[0]].item() == 1234.5 and (pb.state.shares[bad[0]] == want).all()
    ids = np.array([0, 4, 5, 7, E - 3, E - 1])
    teacher = tr.action[:20].index_select(1, torch.as_tensor(ids, device="cuda")).cpu().numpy()
    out = oracle_replay(cfg, mk, params, t0[ids], ids, SEED, 20, teacher, cfg.envs_per_agent)
    compare_rollout(cfg, pb, out, ids, 20)


@pytest.mark.parametrize("name,n,I,hidden,dtype,kernel", [
    ("nasdaq100", 100, 8, (256, 256), "bf16", 1), ("tiny", 5, 4, (1028, 64), "f32", GENERIC),
    ("tiny", 5, 4, (512, 128), "bf16", GENERIC), ("tiny", 5, 4, (64, 64), "f32", FOUR),
    ("tiny", 33, 3, (256, 128), "bf16", FOUR),
])
def test_time_index_at_the_end_of_its_range(name, n, I, hidden, dtype, kernel):
    """t + L past the largest int64 is no room either (the sum must not wrap)."""
    cfg = W.get_config(name).with_(name="last", n=n, n_ind=I, hidden=hidden, dtype=dtype, N=780,
                                   E=9, L=20)
    pb, _ = build_problem(cfg, W.make_market(cfg), np.zeros(9, np.int64))
    assert tp.rollout_kernel(pb.mkt, pb.actor) == kernel
    pb.state = tp.StateT.empty(9, n, count_invalid=True)
    pb.reset()
    far = [2 ** 63 - 1, 2 ** 63 - 20]
    pb.state.t[2], pb.state.t[7] = far
    say(f"[rollout] time indices past the market, {n} stocks {hidden} {dtype}")
    pb.rollout(SEED, 0, 20)
    torch.cuda.synchronize()
    assert pb.state.n_invalid.item() == 2 and pb.state.t[[2, 7]].tolist() == far
    assert torch.isnan(pb.traj.reward[:20, [2, 7]]).all()
    assert torch.isfinite(pb.traj.reward[:20, [0, 1, 3, 4, 5, 6, 8]]).all()


def test_rollout_errors():
    cfg = W.get_config("tiny")
    mk = W.make_market(cfg)
    pb, _ = build_problem(cfg, mk, W.make_t0(cfg))
    with pytest.raises(tp.TPError) as ei:
        pb.rollout(SEED, 200, 100)          # beyond the horizon
    assert ei.value.code == tp.TP_ERANGE
    other = tp.TrajT.alloc(10, cfg.E, cfg.n, cfg.K_pad, torch.float32)
    bad = tp.TrajT(other.action, other.logp, other.reward, other.done,
                   other.obs, 33)           # ld_obs not a multiple of 8
    with pytest.raises(tp.TPError) as ei:
        pb.rollout(SEED, 0, 10, traj=bad)
    assert ei.value.code == tp.TP_EINVAL and "ld_obs" in str(ei.value)


def _one_bar(n, I, h):
    """One bar of 1,024 envs with an fp32 actor, each at a market row of its own:
    the problem, the actor's parameters and its mean in 64 bits."""
    cfg = W.get_config("tiny").with_(name=f"bar-{n}-{h}", n=n, n_ind=I, hidden=(h, h), E=1024,
                                     N=1100)
    mk = W.make_market(cfg)
    pb, (Wl, b, _) = build_problem(cfg, mk, np.arange(1024, dtype=np.int64))
    pb.reset()
    say(f"[rollout] one bar {n} {I} {h}")
    pb.rollout(SEED, 0, 1)
    torch.cuda.synchronize()
    x = pb.traj.obs[0, :, :cfg.S].double().cpu().numpy()
    w = [v[0].astype(np.float64) for v in Wl]
    c = [v[0].astype(np.float64) for v in b]
    return pb, np.tanh(np.tanh(x @ w[0].T + c[0]) @ w[1].T + c[1]) @ w[2].T + c[2]


def _rel2(x, y):
    return float(np.linalg.norm(np.asarray(x, np.float64) - y) / np.linalg.norm(y))


def test_narrow_fp32_actor_against_64_bits():
    """301-32-32-30 fp32: sums of 301 and 32 products.  With m partial sums a
    sum of K products is rounded K / m times at a size that grows with the
    sum, so its error falls as 1 / sqrt(m): measured 1.36e-7 with four,
    1.08e-7 with eight."""
    pb, mu = _one_bar(30, 8, 32)
    e = _rel2(pb.traj.mu_tap[0].cpu().numpy(), mu)
    say(f"    mu {e:.3e}")
    assert e <= 1.2e-7


def test_normals_and_log_density_against_64_bits():
    """The normals' log-density of 30 stocks: fp32 rounds the result (a relative
    2.5e-8 in the 2-norm for values in [2^5, 2^6)) and each of the 30 normals
    (1.5e-8 with correctly rounded ones), together 2.9e-8; a logarithm that is
    2.6e-8 too small on average takes it to 3.5e-8."""
    import oracle
    pb, mu = _one_bar(30, 8, 64)
    key = (SEED & 0xFFFFFFFF, SEED >> 32)
    w = np.array([[oracle.philox((k, e, 0, 0), key) for k in range(8)] for e in range(1024)])
    u = ((w.astype(np.int64) >> 9) + 0.5) * 2.0 ** -23
    rad, ang = np.sqrt(-2 * np.log(u[..., 0::2])), 2 * np.pi * u[..., 1::2]
    z = np.stack([rad * np.cos(ang), rad * np.sin(ang)], -1).reshape(1024, -1)[:, :30]
    ls = float(pb.actor.log_std[0, 0])
    logp = (-0.5 * z * z - ls).sum(1) - 15 * np.log(2 * np.pi)
    e = _rel2(pb.traj.logp[0].cpu().numpy(), logp)
    a = _rel2(pb.traj.action[0].cpu().numpy(), mu + np.exp(ls) * z)
    say(f"    logp {e:.3e} action {a:.3e}")
    assert e <= 3.0e-8 and a <= 1.1e-7


def test_infinite_indicator_at_widths_inside_a_tile():
    """An infinite indicator saturates the first hidden layer (+-1) and nothing
    else: outputs that pad the four-env kernel's layers to whole tiles stay
    out."""
    c = W.get_config("tiny").with_(hidden=(36, 20), N=11, E=8)
    mk = W.make_market(c)
    mk.ind[4, 2, 1], mk.ind[6, 0, 0] = np.inf, -np.inf
    t0 = W.make_t0(c)
    pb, params = build_problem(c, mk, t0)
    pb.reset()
    say("[rollout] infinite indicators")
    pb.rollout(SEED, 0, 10)
    torch.cuda.synchronize()
    teacher = pb.traj.action[:10].cpu().numpy()
    out = oracle_replay(c, mk, params, t0, np.arange(8), SEED, 10, teacher, c.envs_per_agent)
    assert np.isfinite(out["mu"]).all()
    compare_rollout(c, pb, out, np.arange(8), 10)
