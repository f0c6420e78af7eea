"""Host decisions of the library on a CPU: a subprocess loads launch_recorder.c
(a HIP runtime without a device) before libddppo.so and returns what the
library launched.  Runs without torch, whose own HIP runtime would take part."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r'''
import ctypes as C, dataclasses, importlib.util, json, os, sys
sys.path.insert(0, ROOT)
rec = C.CDLL(RECORDER, mode=C.RTLD_GLOBAL)
rec.rec_name.restype, rec.rec_grid_x.restype = C.c_char_p, C.c_uint32
spec = importlib.util.spec_from_file_location("ddppo_lib", os.path.join(ROOT, "paper_1911_00357_amd", "_lib.py"))
L = importlib.util.module_from_spec(spec); spec.loader.exec_module(L)
lib = L.lib()
FAKE = C.c_void_p(1 << 20)      # a device pointer: passed on, never read

def net(dtype="bf16", **kw):
    f = dict(in_ch=4, in_hw=256, avgpool=1, trunk=L.PPO_TRUNK_RESNET, base_width=32, gn_groups=16, compress_ch=128,
             vis_hidden=16, goal_mode=L.PPO_GOAL_POLAR, goal_dim=8, prev_act_dim=8, lstm_layers=1, hidden=64,
             num_actions=4, dtype={"f32": L.PPO_F32, "bf16": L.PPO_BF16}[dtype], cardinality=16, se_reduction=16)
    tiny, blocks = kw.pop("tiny_ch", (32, 128)), kw.pop("blocks", (1, 1, 1, 1))
    f.update(kw)
    d, h = L.NetDesc(**f), C.c_void_p()
    d.tiny_ch[:], d.blocks[:] = tiny, blocks
    L.check(lib.ppo_net_create(C.byref(d), C.byref(h)), "ppo_net_create")
    return h

def launches():
    return [(rec.rec_name(i).decode(), rec.rec_grid_x(i)) for i in range(rec.rec_count())]

def act(h, batch):
    io = L.ActIO(batch=batch)
    for f in ("obs goal prev_action mask h_in c_in u params params_lp action logp value h_out c_out").split():
        setattr(io, f, FAKE)
    rec.rec_reset()
    L.check(lib.ppo_act(h, C.byref(io), FAKE, 1 << 62, None), "ppo_act")
    return launches()

def loss_backward(h, frames):
    nb = min(256, frames)
    lens = (C.c_int32 * nb)(*[frames // nb + (i < frames % nb) for i in range(nb)])
    ids = (C.c_int32 * nb)(*range(nb))
    b = L.Batch(T=lens[0], N=nb, nb=nb, env_ids=C.cast(ids, L.P_i32), lengths=C.cast(lens, L.P_i32))
    for f in ("obs goal prev_action mask action logp_old adv ret h0 c0 params params_lp").split():
        setattr(b, f, FAKE)
    rec.rec_reset()
    cfg = L.LossCfg(clip=0.2, value_coef=0.5, entropy_coef=0.01)
    L.check(lib.ppo_loss_backward(h, C.byref(b), C.byref(cfg), None, FAKE, FAKE, FAKE, 1 << 62, None), "loss_backward")
    return launches()
'''


def record(tmp_path_factory, code: str, env=None):
    """Runs `code` after PRELUDE and returns the JSON value it assigns to `out`."""
    so = tmp_path_factory.getbasetemp() / "launch_recorder.so"
    if not so.exists():
        src = os.path.join(ROOT, "tests", "launch_recorder.c")
        subprocess.run(["gcc", "-std=c99", "-O1", "-shared", "-fPIC", src, "-o", str(so)], check=True)
    head = f"ROOT, RECORDER = {ROOT!r}, {str(so)!r}\n"
    r = subprocess.run([sys.executable, "-c", head + PRELUDE + code + "\nprint('OUT' + json.dumps(out))"],
                       capture_output=True, text=True, timeout=100, env={**os.environ, **(env or {})})
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.split("OUT", 1)[1])
