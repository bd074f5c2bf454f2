"""Performance cases: calls of the library's public entry points over the sizes it is used at, from one decode step of a few tokens to a batch of thousands, both storage types, weights resident in device memory
and streamed from the host.  Every case is a dict of plain values; `prepare` makes what a program holds before the
call (activations, router, page pool and table, workspace), `run` makes the call.

A page pool is filled with independent normal values: packing only reorders the elements of the weight matrices, so a
pool of such values is the packed form of normal weights.  The pages sit at shuffled slots, as in a pool that
has been in use."""
import math

import torch

import paper_2411_11217_amd as M

KIB, MIB = 1 << 10, 1 << 20

# layer shapes: hidden size, expert FFN size, experts, experts per token, page size
SHAPES = {
    "8x7b": (4096, 14336, 8, 2, 2 * MIB),        # the repository's Mixtral-8x7B shape
    "8x22b": (6144, 16384, 8, 2, 4 * MIB),       # its Mixtral-8x22B shape
    "dbrx": (6144, 10752, 16, 4, 4 * MIB),       # its DBRX shape
    "fine": (2048, 1024, 64, 8, 1 * MIB),        # as many experts as the library takes, each of them small
    "mid": (2048, 4096, 8, 2, 2 * MIB),          # a layer of a smaller model
    "tiny": (256, 512, 8, 2, 64 * KIB),          # the repository's smallest workload
    "small": (1024, 2816, 8, 2, 512 * KIB),      # one that still fits a test machine; 22 column tiles of 128
}
ROUTER_SKEW = ((0, 2.5), (7, -1.9))              # router bias of the skewed workload: 40 % / 1 % of the rows


def _case(name, call, shape, T, dtype="bf16", skew=False):
    return {"name": name, "call": call, "shape": shape, "T": T, "dtype": dtype, "skew": skew}


def listed():
    return [
        # a call whose data is next to nothing: launches, latency and the way through the binding
        _case("tiny_f32_t64", "layer", "tiny", 64, "f32"),
        # decode, a handful of requests in flight; the caller has no workspace (the library's static scratch)
        _case("decode_8x7b_t4", "static", "8x7b", 4),
        # the whole GPU task of a decode step after attention: O projection, norm, layer; a micro-batch of 36
        _case("post_attention_8x7b_t36", "post_attention", "8x7b", 36),
        # and the one before attention: residual, norm, QKV projection, bf16 copy
        _case("pre_attention_8x7b_t100", "pre_attention", "8x7b", 100),
        # decode with a full micro-batch: the weights stream once for 64 rows an expert
        _case("decode_8x7b_t256", "layer", "8x7b", 256),
        # many small experts, few rows each
        _case("fine_t777", "layer", "fine", 777),
        # the stages called one by one, as a program does that puts its own steps between them; 16 experts, top 4
        _case("stages_dbrx_t600", "stages", "dbrx", 600),
        # where weight streaming and arithmetic take equally long, row tiles not full
        _case("ridge_8x7b_t1000", "layer", "8x7b", 1000),
        # single precision at a size where it is the arithmetic that counts
        _case("layer_f32_t700", "layer", "small", 700, "f32"),
        # expert pages in pinned host memory, copied while the experts before are computed
        _case("streamed_mid_t1024", "streamed", "mid", 1024),
        # a large batch: the benchmark's default workload
        _case("batch_8x7b_t4096", "layer", "8x7b", 4096),
        # the largest: one expert with two fifths of the rows
        _case("skew_8x22b_t8192", "layer", "8x22b", 8192, "bf16", True),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "stages", "static", "post_attention", "pre_attention", "f32", "streamed"])
    if kind == "f32":
        shape = rng.choice(["tiny", "small"])
        return {"call": rng.choice(["layer", "stages"]), "shape": shape, "T": _log_uniform(rng, 5, 1100), "dtype": "f32", "skew": False}
    if kind == "streamed":
        return {"call": "streamed", "shape": "mid", "T": _log_uniform(rng, 30, 3000), "dtype": "bf16", "skew": False}
    if kind == "static":                         # what fits the static scratch
        shape = rng.choice(["8x7b", "mid", "fine"])
        return {"call": "static", "shape": shape, "T": _log_uniform(rng, 1, {"8x7b": 250, "mid": 600, "fine": 220}[shape]), "dtype": "bf16", "skew": False}
    if kind in ("post_attention", "pre_attention"):
        return {"call": kind, "shape": rng.choice(["8x7b", "dbrx", "mid"]), "T": _log_uniform(rng, 1, 256 if kind == "post_attention" else 3000),
                "dtype": "bf16", "skew": False}
    shape = rng.choice(["8x7b", "8x22b", "dbrx", "fine", "mid", "small"])
    most = {"8x7b": 8192, "8x22b": 8000, "dbrx": 5000, "fine": 8192, "mid": 8192, "small": 8192}[shape]
    return {"call": kind, "shape": shape, "T": _log_uniform(rng, 1, most), "dtype": "bf16", "skew": kind == "layer" and rng.random() < 0.25}


def _shape(case):
    H, F, E, k, page = SHAPES[case["shape"]]
    return M.make_shape(case["T"], H, F, E, k, case["dtype"], page)


def _qkv_width(H):
    return H + H // 2                            # query heads, and a quarter as many key and value heads each


def prepare(case, seed):
    s = _shape(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = s.torch_dtype

    def normal(shape, std=1.0, dtype=dt):
        t = torch.empty(shape, dtype=dtype, device="cuda")
        return t.normal_(0.0, std, generator=g)

    def pool_of(pages):
        return normal((pages, s.page_bytes // (2 if dt == torch.bfloat16 else 4)), 0.02).view(torch.uint8)

    gu, d = M.pages_required(s)
    n_exp = s.E * (gu + d)
    slots = torch.Generator().manual_seed(seed + 1)
    call = case["call"]
    st = {"call": call, "s": s}

    if call == "pre_attention":
        ls = M.make_linear_shape(s.T, s.H, _qkv_width(s.H), s.page_bytes)
        n = M.linear_pages_required(ls)
        st.update(ls=ls, hidden=normal((s.T, s.H), 2.0, torch.float32), delta=normal((s.T, s.H), 1.0, torch.float32),
                  gamma=1.0 + normal((s.H,), 0.1, torch.float32), table=torch.randperm(n, generator=slots).to(torch.int32).cuda(),
                  pool=pool_of(n))
        return st

    st["x"] = normal((s.T, s.H))
    st["Wr"] = normal((s.E, s.H), 0.02)
    st["bias"] = None
    if case["skew"]:
        st["bias"] = torch.zeros(s.E, dtype=torch.float32)
        for e, v in ROUTER_SKEW:
            st["bias"][e] = v
        st["bias"] = st["bias"].cuda()

    if call == "streamed":
        pages = torch.empty((n_exp, s.page_bytes), dtype=torch.uint8, pin_memory=True)
        pages.copy_(pool_of(n_exp))
        table = torch.arange(n_exp, dtype=torch.int32).reshape(s.E, gu + d)       # as the packer lays them out for copying
        st.update(streamer=M.Streamer(s, pages, table), ws=M.Workspace(s), y=torch.empty((s.T, s.H), dtype=torch.float32, device="cuda"))
        st["ids"] = st["ws"].view("topk_ids")
        return st

    extra = 0
    if call == "post_attention":
        st["o_proj"] = M.make_linear_shape(s.T, s.H, s.H, s.page_bytes)
        extra = M.linear_pages_required(st["o_proj"])
        st.update(hidden=normal((s.T, s.H), 2.0, torch.float32), gamma=1.0 + normal((s.H,), 0.1, torch.float32))
    order = torch.randperm(n_exp + extra, generator=slots).to(torch.int32)
    st["table"] = order[:n_exp].reshape(s.E, gu + d).contiguous().cuda()
    st["o_table"] = order[n_exp:].contiguous().cuda()
    st["pool"] = pool_of(n_exp + extra)
    if call in ("layer", "static"):
        st["y"] = torch.empty((s.T, s.H), dtype=torch.float32, device="cuda")
    if call == "layer":
        st["ws"] = M.Workspace(s)
        st["ids"] = st["ws"].view("topk_ids")
    return st


def run(st):
    s, call = st["s"], st["call"]
    if call == "layer":
        M.moe_layer(s, st["x"], st["Wr"], st["table"], st["pool"], bias=st["bias"], workspace=st["ws"], y=st["y"])
        return {"y": st["y"], "ids": st["ids"]}
    if call == "static":
        return {"y": M.moe_layer_static(s, st["x"], st["Wr"], st["table"], st["pool"], st["y"], bias=st["bias"])}
    if call == "stages":
        ids, w, logits = M.moe_route(s, st["x"], st["Wr"], bias=st["bias"], want_logits=True)
        pm = M.moe_permute(s, ids, x=st["x"], topk_w=w)
        h, out = M.moe_expert_ffn(s, pm["x_perm"], pm["offsets"], st["table"], st["pool"])
        y = M.moe_combine(s, out, pm["row_of"], topk_w=w)
        return {"y": y, "ids": ids, "w": w, "logits": logits, "row_of": pm["row_of"], "h": h, "out": out}
    if call == "streamed":
        M.moe_layer_streamed(st["streamer"], st["x"], st["Wr"], bias=st["bias"], workspace=st["ws"], y=st["y"])
        return {"y": st["y"], "ids": st["ids"]}
    if call == "post_attention":
        hidden_mid, x_moe, y, _ = M.moe_post_attention(s, st["o_proj"], st["x"], st["hidden"], st["o_table"], st["gamma"], 1e-5, st["Wr"],
                                                       st["table"], st["pool"])
        return {"hidden_mid": hidden_mid, "x_moe": x_moe, "y": y}
    hidden, x_norm, qkv, qkv16 = M.moe_pre_attention(st["ls"], st["hidden"], st["delta"], st["gamma"], 1e-5, st["table"], st["pool"])
    return {"hidden": hidden, "x_norm": x_norm, "qkv": qkv, "qkv16": qkv16}


def work(case):
    H, F, E, k, page = SHAPES[case["shape"]]
    T, call = case["T"], case["call"]
    R, b = T * k, 2 if case["dtype"] == "bf16" else 4
    if call == "pre_attention":
        N = _qkv_width(H)
        return {"bytes": 2 * H * N + T * H * (4 + 4 + 4 + 2) + T * N * (4 + 2), "flops": 2 * T * H * N}
    experts = E * (1.0 - (1.0 - k / E) ** T)     # experts that some token goes to, on average
    if call == "streamed":
        experts = E                              # every page crosses the host link
    nbytes = experts * 3 * H * F * b + E * H * b + T * H * (b + 4)
    flops = 6 * R * H * F + 2 * T * H * E
    if call == "layer" or call == "streamed":
        nbytes += 4 * R
    if call == "stages":                         # the intermediates are outputs of their calls
        nbytes += R * (H * b + F * b + H * 4) + 4 * T * E + 12 * R
    if call == "post_attention":
        nbytes += 2 * H * H + T * H * (4 + 4 + 2)
        flops += 2 * T * H * H
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured against float64 on the same inputs (the rounding of h to its storage type included), about four times that.
    # f32: rel 6e-7 (tiny) to 1.3e-6 (small), max 9e-6.  bf16: rel 4e-5 for y and 2e-5 for normalised rows, max 2e-3 for y;
    # a rounded output (h, x_norm, the bf16 copy) may land on the neighbouring number, 2^-7 of its value at most, and twice that is
    # allowed.  A token with two equal logits may be given to the other expert ("differ").
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5, "differ": 1e-3}
    return {"rel": 2e-4, "max": 1.6e-2, "differ": 1e-3}
