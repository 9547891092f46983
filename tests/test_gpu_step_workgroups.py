"""The decode step without a band: its token encoded by workgroups of the decode
launch (few units), by the splits' encoder teams, or by a launch of its own.

Whatever the plan takes, the step must write the bytes of nova_kv_encode at
seq_lens - 1 and return nova_kv_decode_attn over the result.  Every format, both
head sizes; an empty sequence, a first token, lengths at the edges of rounds and
splits, a window; contiguous and paged caches; and replays of a captured call
(the handed-over words carry the captured call's tag, so the last to use them
empties them).  A split that does not find its token's words soon forms them
itself: the same has to hold where they never come, or after one look.

Tolerance: the step attends its token with fp32 probabilities, the decode with
fp16 ones (2^-11 of one token's share): 5e-4 of the row norm."""

import numpy as np
import pytest
import torch

import synth
from helpers import row_errors
from oracle import codec as ocodec

pytestmark = pytest.mark.gpu
SAME_TOL = 5e-4


@pytest.fixture(scope="module")
def nk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2608_04074_amd as nk
    nk._native.lib()
    return nk


def dev(x, dtype):
    return torch.as_tensor(np.ascontiguousarray(x)).to(dtype).cuda()


def bits(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda()


def close(got, ref, what):
    g, r = got.cpu().numpy(), ref.cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all(), what
    err = float(row_errors(g.reshape(-1, g.shape[-1]), r.reshape(-1, r.shape[-1])).max())
    print(f"[parity] {what} worst_rel_diff={err:.3e}", flush=True)
    assert err <= SAME_TOL, what


EDGES = [0, 1, 2, 63, 64, 65, 193, 700]
CASES = [
    # D, query heads per KV head, H, lengths, capacity, block size, window, formats
    (128, 4, 8, EDGES, 700, None, 0, ""),                # capacity not a multiple of 16: decode_vq
    (128, 4, 8, EDGES, 704, None, 0, ""),                # one split per unit
    (128, 4, 2, [1500, 1, 1473], 1504, None, 0, ""),     # several splits, their last one short or empty
    (128, 3, 2, [3000, 2881], 3008, 16, 0, "fp8"),
    (128, 4, 2, EDGES, 704, 32, 64, "ks sq"),
    (128, 1, 4, [40, 900, 512], 1024, 16, 0, "ks"),
    (128, 4, 8, [2300] * 8, 2304, 16, 0, ""),            # a full launch round: teams or two launches
    (128, 4, 8, [9000] * 8, 9008, None, 0, "fp8"),
    (64, 8, 8, EDGES, 704, None, 0, ""),
    (64, 8, 8, EDGES, 704, 16, 128, "fp8"),
    (64, 5, 2, [1, 2000, 1985], 2000, 16, 0, "ks sq"),
    (64, 8, 2, [600, 5000], 5008, None, 0, "sq"),
]


@pytest.fixture
def polls(nk, request):
    """How often a split looks for its token's words, for this thread's calls
    (None: as the library sets it; 0: they never come)."""
    hook = nk._native.lib().nova_kv_test_new_token_polls
    hook(-1 if request.param is None else request.param)
    yield request.param
    hook(-1)


@pytest.mark.parametrize("polls", [None, 0, 1], indirect=True)
@pytest.mark.parametrize("D,gqa,H,lens,cap,bs,window,fmt", CASES)
def test_step_is_append_then_decode(nk, polls, D, gqa, H, lens, cap, bs, window, fmt):
    ks, sq, fp8 = (f in fmt.split() for f in ("ks", "sq", "fp8"))
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H * gqa)
    arr = dict(synth.bench_params(wl))
    for k in ("cb_k", "cb_v"):
        if fp8:
            arr[k] = torch.as_tensor(arr[k]).float().to(torch.float8_e4m3fn).view(torch.uint8)
    if sq:
        arr["cb_v"] = None
    P = nk.NovaKVParams.from_arrays(arr, key_scale=ks, sq_values=sq)
    B, L, rng = len(lens), D // 4, np.random.default_rng(len(fmt) + cap)
    bps = 1 if bs is None else cap // bs
    table = None if bs is None else dev(rng.permutation(B * bps).reshape(B, bps), torch.int32)
    lay = nk.CacheLayout.contiguous(cap) if bs is None else nk.CacheLayout(bs, bps, table)
    shape = (B * bps, H, cap if bs is None else bs)
    ck, cv = (rng.integers(0, 256, shape + (L,), dtype=np.uint8) for _ in range(2))
    hks = ocodec.bf16_bits(np.exp(0.3 * rng.standard_normal(shape)))
    hsq = np.stack([ocodec.bf16_bits(np.full(shape, 0.9)), ocodec.bf16_bits(-1.3 + 0.1 * rng.standard_normal(shape))], -1)
    lens_d = dev(lens, torch.int32)
    kn, vn = (dev(rng.standard_normal((B, H, D)), torch.bfloat16) for _ in range(2))
    q = dev(rng.standard_normal((B, H * gqa, D)), torch.bfloat16)
    sinks = dev(rng.standard_normal(H * gqa), torch.float32)
    out = torch.empty((B, H * gqa, D), dtype=torch.float32, device="cuda")
    ws = torch.zeros(nk.decode_workspace_bytes(P, B, H * gqa, cap), dtype=torch.uint8, device="cuda")
    what = f"step D={D} gqa={gqa} H={H} B={B} cap={cap} block={bs} window={window} {fmt} polls={polls}"

    def pools():
        return dict(k=dev(ck, torch.uint8), v=dev(cv, torch.uint8), ks=bits(hks) if ks else None, sq=bits(hsq) if sq else None)

    def reference():
        two = pools()
        nk.encode(P, lay, kn[:, None], vn[:, None], lens_d - 1, two["k"], two["v"], k_scales=two["ks"], v_sq=two["sq"])
        ref = nk.decode_attn(P, lay, q, two["k"], two["v"], lens_d, cap, window=window, sinks=sinks, k_scales=two["ks"],
                             v_sq=two["sq"])
        return two, ref

    one = pools()

    def step():
        nk.append_decode_attn(P, lay, kn, vn, q, one["k"], one["v"], lens_d, cap, window=window, sinks=sinks, out=out,
                              workspace=ws, k_scales=one["ks"], v_sq=one["sq"])

    print(f"[gpu-case] {what}", flush=True)
    two, ref = reference()
    for _ in range(2):
        step()
    torch.cuda.synchronize()
    for name in ("k", "v", "ks", "sq"):
        if one[name] is not None:
            assert torch.equal(one[name], two[name]), f"{what}: other {name} bytes"
    close(out, ref, what)
    if 0 in lens:
        assert not out[lens.index(0)].any()

    # a captured call, replayed on other inputs with eager work between
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        step()
    for r in range(3):
        kn.copy_(torch.randn_like(kn))
        vn.copy_(torch.randn_like(vn))
        q.copy_(torch.randn_like(q))
        g.replay()
        torch.cuda.synchronize()
        got = out.clone()
        two, ref = reference()
        torch.cuda.synchronize()
        close(got, ref, f"{what} replay {r}")
        assert torch.equal(one["k"], two["k"]) and torch.equal(one["v"], two["v"])
        step()
        torch.cuda.synchronize()


@pytest.mark.parametrize("polls", [None, 0, 1], indirect=True)
@pytest.mark.parametrize("D,lens,cap", [(128, [2000], 2048), (128, [500, 0, 3], 512), (64, [150, 0, 3], 192)])
def test_replay_leaves_no_words(nk, polls, D, lens, cap):
    """Replays of a captured step repeat its tag: each leaves the workspace all
    zero, whether the split took the handed-over words or gave up on them (its
    encoder's words then come later), so none is there for the next one.  (One
    split at head_dim 64, whose split partials are plain words.)"""
    H, gqa, B = 2, 4, len(lens)
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H * gqa)
    P = nk.NovaKVParams.from_arrays(dict(synth.bench_params(wl)))
    rng = np.random.default_rng(cap)
    ck, cv = (dev(rng.integers(0, 256, (B, H, cap, D // 4), dtype=np.uint8), torch.uint8) for _ in range(2))
    kn, vn = (dev(rng.standard_normal((B, H, D)), torch.bfloat16) for _ in range(2))
    q = dev(rng.standard_normal((B, H * gqa, D)), torch.bfloat16)
    lens_d = dev(lens, torch.int32)
    out = torch.empty((B, H * gqa, D), dtype=torch.float32, device="cuda")
    ws = torch.zeros(nk.decode_workspace_bytes(P, B, H * gqa, cap), dtype=torch.uint8, device="cuda")

    def step():
        nk.append_decode_attn(P, nk.CacheLayout.contiguous(cap), kn, vn, q, ck, cv, lens_d, cap, out=out, workspace=ws)

    print(f"[gpu-case] replays of a captured step D={D} lens={lens} polls={polls}", flush=True)
    step()
    torch.cuda.synchronize()
    ref = out.clone()
    ws.zero_()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert not ws.any()
        close(out, ref, f"replayed step D={D} lens={lens}")


@pytest.mark.parametrize("D,fmt,bs,band", [(64, "", None, False), (128, "ks sq", 16, False), (64, "ks", 32, False),
                                           (128, "ks sq", 16, True)])
def test_a_length_past_the_capacity_stores_nothing(nk, D, fmt, bs, band):
    """seq_lens one past a sequence's capacity is a caller's mistake; the step
    stores nothing of that token, as the append does (the rows after the
    sequence's are another's, in bounds of the pools here)."""
    ks, sq = (f in fmt.split() for f in ("ks", "sq"))
    H, gqa, B, cap, L = 2, 4, 3, 192, D // 4
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H * gqa)
    arr = dict(synth.bench_params(wl))
    if sq:
        arr["cb_v"] = None
    P = nk.NovaKVParams.from_arrays(arr, key_scale=ks, sq_values=sq)
    bps = 1 if bs is None else cap // bs
    lay = (nk.CacheLayout.contiguous(cap) if bs is None else
           nk.CacheLayout(bs, bps, torch.arange(B * bps, dtype=torch.int32, device="cuda").reshape(B, bps)))
    shape = (B * bps, H, cap if bs is None else bs)
    rng = np.random.default_rng(D)
    pools = [dev(rng.integers(0, 256, shape + (L,), dtype=np.uint8), torch.uint8) for _ in range(2)]
    pools += [bits(ocodec.bf16_bits(np.ones(shape)))] if ks else [None]
    pools += [bits(ocodec.bf16_bits(np.ones(shape + (2,))))] if sq else [None]
    bnd = nk.Band(4, 16, *(torch.zeros((B, H, 20, D), dtype=torch.bfloat16, device="cuda") for _ in range(2))) if band else None
    kept = pools + ([bnd.k, bnd.v] if band else [])
    before = [None if x is None else x.clone() for x in kept]
    kn, vn = (dev(rng.standard_normal((B, H, D)), torch.bfloat16) for _ in range(2))
    q = dev(rng.standard_normal((B, H * gqa, D)), torch.bfloat16)
    print(f"[gpu-case] step past the capacity D={D} {fmt} block={bs} band={band}", flush=True)
    nk.append_decode_attn(P, lay, kn, vn, q, pools[0], pools[1], dev([cap + 1, 0, 0], torch.int32), cap,
                          k_scales=pools[2], v_sq=pools[3], band=bnd)
    torch.cuda.synchronize()
    for x, y in zip(kept, before):
        assert x is None or torch.equal(x, y)


@pytest.mark.parametrize("D,fmt", [(128, ""), (64, "ks")])
def test_steps_on_several_streams(nk, D, fmt):
    """Four steps in flight at once, each on a stream and a workspace of its own,
    whose encoder and decoding workgroups together are more than the CUs."""
    H, gqa, B, cap, n = 8, 4, 15, 512, 4
    ks = fmt == "ks"
    wl = synth.get_workload("qwen3_8b" if D == 128 else "gptoss_pair").scaled(num_kv_heads=H, num_q_heads=H * gqa)
    P = nk.NovaKVParams.from_arrays(dict(synth.bench_params(wl)), key_scale=ks)
    lay, gen = nk.CacheLayout.contiguous(cap), torch.Generator(device="cuda").manual_seed(D)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    lens = torch.full((B,), 500, dtype=torch.int32, device="cuda")
    jobs = []
    for _ in range(n):
        k, v = (torch.randint(0, 256, (B, H, cap, D // 4), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(2))
        jobs.append(dict(kn=rnd(B, H, D), vn=rnd(B, H, D), q=rnd(B, H * gqa, D), k=k, v=v,
                         sc=torch.ones((B, H, cap), dtype=torch.bfloat16, device="cuda") if ks else None,
                         out=torch.zeros((B, H * gqa, D), device="cuda"), stream=torch.cuda.Stream(),
                         ws=torch.zeros(nk.decode_workspace_bytes(P, B, H * gqa, cap), dtype=torch.uint8, device="cuda")))

    def step(j, stream=None):
        nk.append_decode_attn(P, lay, j["kn"], j["vn"], j["q"], j["k"], j["v"], lens, cap, out=j["out"], workspace=j["ws"],
                              k_scales=j["sc"], stream=stream)

    print(f"[gpu-case] steps on {n} streams D={D} {fmt}", flush=True)
    want = []
    for j in jobs:
        step(j)
        torch.cuda.synchronize()
        want.append([x.clone() for x in (j["out"], j["k"], j["v"])])
    for _ in range(8):
        for j in jobs:
            j["out"].zero_()
        torch.cuda.synchronize()
        for j in jobs:
            step(j, j["stream"])
        torch.cuda.synchronize()
        for j, w in zip(jobs, want):
            close(j["out"], w[0], f"step on a stream D={D} {fmt}")
            assert torch.equal(j["k"], w[1]) and torch.equal(j["v"], w[2])
