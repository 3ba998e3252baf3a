"""GPU parity of tp_critic_value (the PPO critic's forward pass over a
trajectory's observations) against the oracle's MLP: the bf16 MFMA kernel at
512- and 1024-wide layers (one agent and several agents, ragged row blocks),
the tile kernel (fp32 and other bf16 shapes), the full 100-stock minute
trajectory shape on sampled rows, and determinism.

Observation blocks [T][E][K_pad] come from the seeded generator
(workloads.make_learner_data: the observation's structure and scales, zero
padding), rounded to bf16 on the CPU for bf16 critics; both sides read the
same values."""

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_common import TOL_MLP, rel_check, say
from paper_2111_05188_amd import tp

pytestmark = pytest.mark.gpu


def _oracle_critic(cfg, params, A):
    """The critic as an oracle MLP with one output (log_std unused)."""
    Wc, bc = params
    S, H1, H2, _ = cfg.dims
    Wo = [Wc[0], Wc[1], Wc[2].reshape(A, 1, H2)]
    bo = [bc[0], bc[1], bc[2].reshape(A, 1)]
    return oracle.actor(Wo, bo, np.zeros((A, 1), np.float32), (S, H1, H2, 1),
                        cfg.dtype == "bf16", cfg.E // A)


POOL = 65536


def _obs_block(c, T, E, seed):
    """[T][E][K_pad] observation rows of the critic's dtype on the device,
    row r = t E + e holding generated row r mod POOL, and the host values
    of the generated rows (what the oracle reads)."""
    n = min(T * E, POOL)
    obs, *_ = W.make_learner_data(c, n, seed=seed)
    base = torch.from_numpy(obs)
    if c.dtype == "bf16":
        base = base.to(torch.bfloat16)
    host = base.float().numpy()
    dev = base.cuda()
    sel = torch.arange(T * E, device="cuda") % n
    return dev.index_select(0, sel).reshape(T, E, c.K_pad), host


def _run(cfg, E, L, n_agents=1, sample=None):
    c = cfg.with_(E=E, n_agents=n_agents, L=L)
    T1 = L + 1
    obs_all, host = _obs_block(c, T1, E, seed=E * 7 + L)
    cp = W.make_critic(c)
    dt = tp.TP_BF16 if c.dtype == "bf16" else tp.TP_F32
    crit = tp.CriticT([torch.from_numpy(w).cuda() for w in cp[0]],
                      [torch.from_numpy(x).cuda() for x in cp[1]], c.dims[:3], dt,
                      E // n_agents)
    crit.pack()
    values = torch.empty(T1, E, dtype=torch.float32, device="cuda")
    say(f"[critic] {cfg.name} E={E} T={T1} agents={n_agents}")
    tp.critic_value(crit, obs_all, values)
    torch.cuda.synchronize()
    v = values.cpu().numpy()                          # [L+1][E]
    act = _oracle_critic(c, cp, n_agents)
    epa = E // n_agents
    if sample is None:
        rows_ = [(t, e) for t in range(T1) for e in range(E)]
    else:
        rng = np.random.default_rng(5)
        rows_ = [(int(rng.integers(T1)), int(rng.integers(E))) for _ in range(sample)]
    got, want = [], []
    for a in range(n_agents):
        sel = [(t, e) for (t, e) in rows_ if e // epa == a]
        if not sel:
            continue
        x = host[[(t * E + e) % host.shape[0] for t, e in sel], :c.S]
        want.append(oracle.mlp(act, a, x)[:, 0])
        got.append(np.array([v[t, e] for t, e in sel]))
    got, want = np.concatenate(got), np.concatenate(want)
    rel_check(f"critic {cfg.name}", got, want, TOL_MLP[c.dtype])
    return crit, obs_all, values


def test_critic_mfma_512_ragged():
    # 1001-512-512-1 bf16: 300 envs = two 128-row blocks and a ragged 44
    _run(W.get_config("nasdaq100"), 300, 6)


def test_critic_mfma_1024():
    _run(W.get_config("stress"), 70, 4)


def test_critic_mfma_three_agents():
    # agent blocks of 45 envs: every block of rows stays inside one agent
    _run(W.get_config("ensemble"), 135, 5, n_agents=3)


@pytest.mark.parametrize("name", ["nasdaq100", "stress"])
def test_critic_mfma_few_envs_per_agent(name):
    # two envs an agent: a block of rows spans 32 or 64 steps, the last one ragged
    _run(W.get_config(name), 6, 70, n_agents=3)


def test_critic_generic_fp32():
    _run(W.get_config("tiny"), 40, 30)
    _run(W.get_config("dow30"), 33, 20)


def test_critic_generic_bf16_other_shape():
    _run(W.get_config("dow30").with_(dtype="bf16"), 33, 20)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,hidden,E,L,A", [
    (5, (4, 4), 1, 1, 1),             # one row; widths below a tile, one k-block
    (7, (36, 100), 21, 11, 3),        # seven envs an agent: tiles span steps; ragged widths
    (5, (260, 268), 90, 99, 2),       # more than one round of tiles: both row buffers
    (5, (64, 48), 700, 60, 1),        # the largest row tile, a ragged last one
    (30, (256, 256), 130, 130, 1),    # two row tiles of fp32, four of bf16
])
def test_critic_tile_kernel_edges(n, hidden, E, L, A, dtype):
    cfg = W.get_config("tiny").with_(name=f"tile-{hidden}", n=n, n_ind=8, hidden=hidden,
                                     dtype=dtype)
    _run(cfg, E, L, n_agents=A, sample=None if E * L < 4000 else 500)


def test_critic_ignores_columns_past_the_state():
    """Columns S .. K_pad of the rows are ignored, whatever they hold."""
    cfg = W.get_config("tiny").with_(hidden=(32, 32))
    crit, obs, values = _run(cfg, 40, 3)
    v0 = values.clone()
    obs = obs.clone()
    obs[:, :, cfg.S:] = float("nan")
    tp.critic_value(crit, obs, values)
    torch.cuda.synchronize()
    assert torch.equal(v0, values)


def test_critic_full_nasdaq_trajectory_sampled():
    cfg = W.get_config("nasdaq100")
    crit, obs_all, values = _run(cfg, cfg.E, cfg.L, sample=256)
    # determinism: a second call gives the same bits
    v0 = values.clone()
    tp.critic_value(crit, obs_all, values)
    torch.cuda.synchronize()
    assert torch.equal(v0, values)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tanh_of_the_tile_kernel(dtype):
    """The hidden layers' tanh, read through a critic that passes one input
    on: h1 = tanh(x), then a second layer whose input is scaled by 2^-20 (its
    tanh is its argument, to 2^-40) and a head of 2^20, so V = tanh(x).

    fp32: within 1 ulp of tanh (measured over every fp32 value: 0.975; the
    library's tanhf reaches 1.41).  bf16: half a bf16 ulp and what the fp32
    error before the rounding adds, 1.35 * 2^-16 of one."""
    k = torch.arange(2 ** 20, dtype=torch.float64, device="cuda")
    x = torch.cat([12.0 * (k + 0.5) / 2 ** 20, 2.0 ** (-40 + 40 * k / 2 ** 20),
                   torch.tensor([0.0, 1.0, 10.0, 1e30], dtype=torch.float64, device="cuda")])
    x = torch.cat([x, -x]).float()
    bf = dtype == "bf16"
    if bf:
        x = x.bfloat16().float()
    W1, W2, w3 = torch.zeros(1, 4, 1), torch.zeros(1, 4, 4), torch.zeros(1, 4)
    W1[0, 0, 0], W2[0, 0, 0], w3[0, 0] = 1.0, 2.0 ** -20, 2.0 ** 20
    b = [torch.zeros(1, 4).cuda(), torch.zeros(1, 4).cuda(), torch.zeros(1).cuda()]
    crit = tp.CriticT([W1.cuda(), W2.cuda(), w3.cuda()], b, (1, 4, 4),
                      tp.TP_BF16 if bf else tp.TP_F32, 1024)
    crit.pack()
    T = -(-x.numel() // 1024)
    rows = torch.zeros(T * 1024, 32, device="cuda")
    rows[:x.numel(), 0] = x
    rows = rows.view(T, 1024, 32)
    value = torch.empty(T, 1024, device="cuda")
    say(f"[critic] tanh {dtype}")
    tp.critic_value(crit, rows.bfloat16() if bf else rows, value)
    torch.cuda.synchronize()
    got, want = value.view(-1)[:x.numel()].double(), torch.tanh(x.double())
    ulp = torch.exp2(torch.floor(torch.log2(want.abs().clamp(min=2.0 ** -126))) - (7 if bf else 23))
    err = ((got - want).abs() / ulp).max().item()
    say(f"    worst error {err:.4f} ulp of {dtype}")
    assert err <= (0.5 + 1.35 * 2.0 ** -16 if bf else 1.0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_input_at_widths_inside_a_tile(dtype):
    """An infinite observation saturates the first hidden layer (+-1) and
    nothing else: columns that pad the layers to whole tiles stay out."""
    cfg = W.get_config("tiny").with_(hidden=(36, 20), dtype=dtype, E=24, L=2, n_agents=1)
    obs, host = _obs_block(cfg, 3, 24, seed=3)
    obs, host = obs.clone(), host.copy()
    obs[1, 5, 7], obs[2, 9, cfg.S - 1] = float("inf"), float("-inf")
    host[24 + 5, 7], host[48 + 9, cfg.S - 1] = np.inf, -np.inf
    cp = W.make_critic(cfg)
    crit = tp.CriticT([torch.from_numpy(w).cuda() for w in cp[0]],
                      [torch.from_numpy(x).cuda() for x in cp[1]], cfg.dims[:3],
                      tp.TP_BF16 if dtype == "bf16" else tp.TP_F32, 24)
    crit.pack()
    value = torch.empty(3, 24, device="cuda")
    say(f"[critic] infinite inputs {dtype}")
    tp.critic_value(crit, obs, value)
    torch.cuda.synchronize()
    want = oracle.mlp(_oracle_critic(cfg, cp, 1), 0, host[:72, :cfg.S])[:, 0]
    assert np.isfinite(want).all()
    rel_check("values", value.view(-1).cpu().numpy(), want, TOL_MLP[dtype])
