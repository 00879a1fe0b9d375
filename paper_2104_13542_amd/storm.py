"""Python binding of the HIP library ``libstorm.so`` (ctypes).

Argument marshalling only: tensors are allocated with torch on the current
HIP device, their device pointers and the current stream are handed to the C
ABI declared in ``include/storm.h``, and every step of the MPC iteration runs
in the library's kernels.  There is no fallback: if the library has not been
built, importing this module raises.
"""
from __future__ import annotations

import ctypes
import os

import numpy as np
import torch

from . import inputs

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libstorm.so")

DOF = 7
NTERMS = 9
TERM_NAMES = ("pos", "rot", "joint", "vel", "stop", "manip", "self", "env")

STORM_OK = 0
STORM_E_NULL = -1
STORM_E_RANGE = -2
STORM_E_PARAM = -3
STORM_E_DEVICE = -4
STORM_E_STATE = -5
STORM_E_NOMEM = -6
STORM_E_UNSUPPORTED = -7
FLAG_NONFINITE_COST = 1
FLAG_ZERO_WEIGHT = 2


class StormError(RuntimeError):
    def __init__(self, code, where):
        self.code = code
        super().__init__("%s: %s (%d)" % (where, status_str(code), code))


class storm_params(ctypes.Structure):
    _fields_ = [
        ("n_particles", ctypes.c_int32), ("horizon", ctypes.c_int32), ("n_halton", ctypes.c_int32),
        ("n_null", ctypes.c_int32), ("n_knots", ctypes.c_int32), ("cost_mask", ctypes.c_uint32),
        ("seed", ctypes.c_uint64), ("dt", ctypes.POINTER(ctypes.c_float)),
        ("sigma_init", ctypes.c_float * 7),
        ("beta", ctypes.c_float), ("gamma", ctypes.c_float), ("alpha_mu", ctypes.c_float),
        ("alpha_sigma", ctypes.c_float), ("w_term", ctypes.c_float), ("sigma2_min", ctypes.c_float),
        ("acc_stop", ctypes.c_float), ("k_jl", ctypes.c_float), ("k_vl", ctypes.c_float), ("k_m", ctypes.c_float),
        ("w_pos", ctypes.c_float), ("w_rot", ctypes.c_float),
        ("alpha_pos", ctypes.c_float * 3), ("alpha_rot", ctypes.c_float * 3),
        ("a_stop", ctypes.c_float), ("a_joint", ctypes.c_float), ("a_vel", ctypes.c_float),
        ("a_manip", ctypes.c_float), ("a_coll", ctypes.c_float), ("grad_mask", ctypes.c_uint32),
        ("comb_filter", ctypes.c_int32), ("comb", ctypes.c_float * 3), ("cov_per_step", ctypes.c_int32),
        ("w_ball", ctypes.c_float), ("ball_gravity", ctypes.c_float * 3), ("ball_center", ctypes.c_float * 2),
        ("self_model", ctypes.c_int32),
    ]


class storm_robot(ctypes.Structure):
    _fields_ = [
        ("dh", (ctypes.c_float * 3) * 8),
        ("q_min", ctypes.c_float * 7), ("q_max", ctypes.c_float * 7), ("qd_max", ctypes.c_float * 7),
        ("n_spheres", ctypes.c_int32), ("spheres", ctypes.POINTER(ctypes.c_float)),
        ("self_mlp", ctypes.POINTER(ctypes.c_float)),
    ]


class storm_scene(ctypes.Structure):
    _fields_ = [("n_obstacles", ctypes.c_int32), ("obstacles", ctypes.POINTER(ctypes.c_float))]


class storm_debug(ctypes.Structure):
    _fields_ = [(k, ctypes.c_void_p) for k in ("u", "q", "v", "a", "c", "terms", "xd", "xdd")]


_lib = None

# every symbol declared in include/storm.h
EXPORTS = (
    "storm_rollout_init", "storm_rollout_step", "storm_rollout_update", "storm_rollout_destroy",
    "storm_rollout_status", "storm_rollout_get_state", "storm_rollout_set_state", "storm_fk",
    "storm_status_str", "storm_rollout_graph_create", "storm_rollout_graph_launch", "storm_rollout_graph_destroy",
    "storm_batch_init", "storm_batch_step", "storm_batch_update", "storm_batch_graph_create",
    "storm_batch_set_config", "storm_batch_get_config", "storm_batch_autotune", "storm_batch_get_state",
    "storm_batch_set_state", "storm_batch_costs", "storm_batch_destroy", "storm_plant_step",
    "storm_rollout_grad", "storm_rollout_grad_noalloc", "storm_rollout_refine", "storm_rollout_graph_create_refine",
    "storm_batch_refine", "storm_batch_graph_create_refine", "storm_rollout_set_ball", "storm_rollout_control",
    "storm_fk_rows",
)


class storm_launch_config(ctypes.Structure):
    _fields_ = [("waves", ctypes.c_int32), ("grid", ctypes.c_int32), ("cost_order", ctypes.c_int32)]


def lib():
    """Load libstorm.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError("libstorm.so is not built (run paper_2104_13542_amd.build.build())")
        L = ctypes.CDLL(LIB_PATH)
        vp = ctypes.c_void_p
        i32 = ctypes.c_int32
        L.storm_status_str.argtypes = [i32]
        L.storm_status_str.restype = ctypes.c_char_p
        L.storm_rollout_init.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(storm_params),
                                         ctypes.POINTER(storm_robot), ctypes.POINTER(storm_scene), vp]
        L.storm_rollout_step.argtypes = [vp, vp, vp, vp, ctypes.POINTER(storm_debug), vp, vp]
        L.storm_rollout_update.argtypes = [vp, vp, vp, vp, i32, vp]
        L.storm_rollout_control.argtypes = [vp, vp, vp, vp, i32, i32, vp]
        L.storm_rollout_set_ball.argtypes = [vp, vp, vp]
        L.storm_rollout_destroy.argtypes = [vp]
        L.storm_rollout_status.argtypes = [vp, ctypes.POINTER(ctypes.c_uint32), vp]
        L.storm_rollout_get_state.argtypes = [vp, vp, vp, vp, vp]
        L.storm_rollout_set_state.argtypes = [vp, vp, vp, vp, vp]
        L.storm_fk.argtypes = [ctypes.POINTER(storm_robot), vp, i32, vp, vp, vp]
        L.storm_fk_rows.argtypes = L.storm_fk.argtypes
        L.storm_rollout_graph_create.argtypes = [vp, vp, vp, vp, i32, i32, vp, ctypes.POINTER(vp)]
        L.storm_rollout_graph_launch.argtypes = [vp, vp]
        L.storm_rollout_graph_destroy.argtypes = [vp]
        L.storm_batch_init.argtypes = [ctypes.POINTER(vp), i32, ctypes.POINTER(storm_params),
                                       ctypes.POINTER(storm_robot), ctypes.POINTER(storm_scene), vp]
        L.storm_batch_step.argtypes = [vp, vp, vp, vp]
        L.storm_batch_update.argtypes = [vp, vp, i32, vp]
        L.storm_batch_graph_create.argtypes = [vp, vp, vp, vp, i32, i32, vp, ctypes.POINTER(vp)]
        L.storm_batch_set_config.argtypes = [vp, ctypes.POINTER(storm_launch_config)]
        L.storm_batch_get_config.argtypes = [vp, ctypes.POINTER(storm_launch_config)]
        L.storm_batch_autotune.argtypes = [vp, vp, vp, i32, vp, ctypes.POINTER(storm_launch_config), vp,
                                           ctypes.POINTER(i32)]
        L.storm_batch_get_state.argtypes = [vp, i32, vp, vp, vp, vp]
        L.storm_batch_set_state.argtypes = [vp, i32, vp, vp, vp, vp]
        L.storm_batch_costs.argtypes = [vp, i32, vp, vp]
        L.storm_batch_destroy.argtypes = [vp]
        L.storm_plant_step.argtypes = [vp, vp, i32, ctypes.c_float, vp]
        L.storm_rollout_grad.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp]
        L.storm_rollout_grad_noalloc.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp]
        L.storm_rollout_refine.argtypes = [vp, vp, vp, i32, ctypes.c_float, vp, i32, vp]
        L.storm_rollout_graph_create_refine.argtypes = [vp, vp, vp, vp, i32, i32, i32, ctypes.c_float, vp,
                                                        ctypes.POINTER(vp)]
        L.storm_batch_refine.argtypes = [vp, vp, vp, i32, ctypes.c_float, vp, i32, vp]
        L.storm_batch_graph_create_refine.argtypes = [vp, vp, vp, vp, i32, i32, i32, ctypes.c_float, vp,
                                                      ctypes.POINTER(vp)]
        for name in EXPORTS:
            getattr(L, name).restype = ctypes.c_char_p if name == "storm_status_str" else i32
        _lib = L
    return _lib


def status_str(code):
    return lib().storm_status_str(int(code)).decode()


def _check(code, where):
    if code != STORM_OK:
        raise StormError(code, where)


def _ptr(t):
    # an int: the functions' argument types make the pointer of it
    return t.data_ptr() if t is not None else None


def _stream():
    # the raw handle of the current stream, without building a Stream object
    # or asking for the device through torch.cuda's checks (every caller holds
    # a context or a tensor of the device)
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def make_params(p: "inputs.Params"):
    """Fill a storm_params from an inputs.Params; returns (struct, keep-alive)."""
    sp = storm_params()
    sp.n_particles, sp.horizon = p.n_particles, p.horizon
    sp.n_halton, sp.n_null, sp.n_knots = p.n_halton, p.n_null, p.n_knots
    sp.cost_mask, sp.seed = p.cost_mask, p.seed
    sp.grad_mask = getattr(p, "grad_mask", 0)
    sp.comb_filter = int(getattr(p, "comb_filter", 0))
    sp.cov_per_step = int(getattr(p, "cov_per_step", 0))
    sp.w_ball = float(getattr(p, "w_ball", 0.0))
    sp.self_model = int(getattr(p, "self_model", 0))
    for c, g in enumerate(getattr(p, "ball_gravity", (0.0, 0.0, -9.81))):
        sp.ball_gravity[c] = float(g)
    for c, x in enumerate(getattr(p, "ball_center", (0.0, 0.0))):
        sp.ball_center[c] = float(x)
    comb = getattr(p, "comb", (1.0, 0.0, 0.0))
    for c in range(3):
        sp.comb[c] = float(comb[c])
    dt = np.ascontiguousarray(p.dt, dtype=np.float32)
    sp.dt = dt.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    for j in range(DOF):
        sp.sigma_init[j] = float(p.sigma_init[j])
    for k in ("beta", "gamma", "alpha_mu", "alpha_sigma", "w_term", "sigma2_min", "acc_stop", "k_jl", "k_vl",
              "k_m", "w_pos", "w_rot", "a_stop", "a_joint", "a_vel", "a_manip", "a_coll"):
        setattr(sp, k, float(getattr(p, k)))
    for c in range(3):
        sp.alpha_pos[c] = float(p.alpha_pos[c])
        sp.alpha_rot[c] = float(p.alpha_rot[c])
    return sp, dt


def make_robot(spheres=None, dh=None, q_min=None, q_max=None, qd_max=None, self_mlp=None):
    """storm_robot for the Panda (or the given DH and limits); self_mlp: the
    learned self-collision network's parameters [STORM_SELF_MLP_SIZE]."""
    # the Panda in one go (the struct begins with its floats: dh, q_min, q_max,
    # qd_max), then what is given, element by element
    flat = np.zeros(ctypes.sizeof(storm_robot) // 4, dtype=np.float32)
    flat[:24].reshape(8, 3)[:] = inputs.PANDA_DH
    for k, limits in enumerate((inputs.PANDA_Q_MIN, inputs.PANDA_Q_MAX, inputs.PANDA_QD_MAX)):
        flat[24 + DOF * k:24 + DOF * (k + 1)] = limits
    r = storm_robot.from_buffer_copy(flat)
    if dh is not None:
        for k in range(8):
            for c in range(3):
                r.dh[k][c] = float(dh[k][c])
    for field, given in ((r.q_min, q_min), (r.q_max, q_max), (r.qd_max, qd_max)):
        if given is not None:
            for j in range(DOF):
                field[j] = float(given[j])
    sph = np.ascontiguousarray(np.zeros((0, 5)) if spheres is None else spheres, dtype=np.float32)
    r.n_spheres = sph.shape[0]
    r.spheres = sph.ctypes.data_as(ctypes.POINTER(ctypes.c_float)) if sph.size else None
    if self_mlp is not None:
        mlp = np.ascontiguousarray(self_mlp, dtype=np.float32)
        r.self_mlp = mlp.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
        r._self_mlp = mlp  # kept alive with the struct
    return r, sph


def make_scene(obstacles):
    s = storm_scene()
    obs = np.ascontiguousarray(obstacles.reshape(-1, inputs.OBSTACLE_STRIDE), dtype=np.float32)
    s.n_obstacles = obs.shape[0]
    s.obstacles = obs.ctypes.data_as(ctypes.POINTER(ctypes.c_float)) if obs.size else None
    return s, obs


class Rollout:
    """One MPC problem on the current HIP device (plain form)."""

    def __init__(self, problem: "inputs.Problem", device=None):
        self.device = torch.device("cuda") if device is None else torch.device(device)
        self.problem = problem
        p = problem.params
        self.N, self.H = p.n_particles, p.horizon
        sp, self._dt = make_params(p)
        rb, self._sph = make_robot(problem.spheres, self_mlp=getattr(problem, "self_mlp", None))
        sc, self._obs = make_scene(problem.obstacles)
        self._robot = rb
        handle = ctypes.c_void_p()
        torch.cuda.init()
        with torch.cuda.device(self.device):
            _check(lib().storm_rollout_init(ctypes.byref(handle), ctypes.byref(sp), ctypes.byref(rb),
                                            ctypes.byref(sc), _stream()), "storm_rollout_init")
        self._h = handle
        self.x0 = torch.tensor(np.concatenate([problem.q0, problem.v0, problem.a0]), dtype=torch.float32,
                               device=self.device)
        self.cmd = torch.zeros(DOF, dtype=torch.float32, device=self.device)
        # what new outputs are shaped like (an allocation like another tensor
        # costs less host time than one from a shape)
        self._mean_like = torch.empty((self.H, DOF), dtype=torch.float32, device=self.device)
        self._sigma2_like = torch.empty(self._sig_shape(), dtype=torch.float32, device=self.device)

    # -- lifecycle ---------------------------------------------------------
    def close(self):
        if getattr(self, "_h", None) is not None and self._h.value:
            lib().storm_rollout_destroy(self._h)
            self._h = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    # -- MPC iteration -----------------------------------------------------
    def step(self, goal, x0=None, noise=None, debug=False, C=None, task_space=False):
        """Sample + roll out.  goal: [12] device tensor.  noise: optional
        [7][N][H] standard normals.  task_space: also return the flange
        velocity and acceleration xd, xdd [6][N][H] (Eq. 8).  Returns a dict
        of the requested outputs."""
        N, H = self.N, self.H
        x0 = self.x0 if x0 is None else x0
        out = {}
        dbg = None
        if debug:
            kw = dict(dtype=torch.float32, device=self.device)
            for k in ("u", "q", "v", "a"):
                out[k] = torch.empty((DOF, N, H), **kw)
            out["c"] = torch.empty((N, H), **kw)
            out["terms"] = torch.empty((NTERMS, N, H), **kw)
            dbg = storm_debug(*[out[k].data_ptr() for k in ("u", "q", "v", "a", "c", "terms")])
        if task_space:
            if dbg is None:
                dbg = storm_debug()
            for k in ("xd", "xdd"):
                out[k] = torch.empty((6, N, H), dtype=torch.float32, device=self.device)
                setattr(dbg, k, out[k].data_ptr())
        if C is None:
            C = torch.empty(N, dtype=torch.float32, device=self.device)
        out["C"] = C
        _check(lib().storm_rollout_step(self._h, _ptr(x0), _ptr(goal), _ptr(noise),
                                        ctypes.byref(dbg) if dbg is not None else None, _ptr(C), _stream()),
               "storm_rollout_step")
        return out

    def set_ball(self, ball):
        """The ball's world-frame position and velocity [6] (device tensor)
        at the current arm state, for the ball term."""
        ball = ball.contiguous()
        _check(lib().storm_rollout_set_ball(self._h, _ptr(ball), _stream()), "storm_rollout_set_ball")
        self._ball = ball  # kept alive until the copy has run

    def _sig_shape(self):
        return (self.H, DOF) if getattr(self.problem.params, "cov_per_step", 0) else (DOF,)

    def update(self, shift=True, want_mean=True, cmd=None):
        """Policy update; returns (cmd [7], mean' [H][7] or None, sigma2' [7]
        ([H][7] with cov_per_step) or None)."""
        mean = torch.empty_like(self._mean_like) if want_mean else None
        sigma2 = torch.empty_like(self._sigma2_like) if want_mean else None
        cmd = self.cmd if cmd is None else cmd
        _check(lib().storm_rollout_update(self._h, _ptr(mean), _ptr(sigma2), _ptr(cmd), int(bool(shift)),
                                          _stream()), "storm_rollout_update")
        return cmd, mean, sigma2

    def control(self, x0, goal, cmd, iterations=1, shift=True):
        """One whole control step (Alg. 1) in one call: `iterations` rounds
        of step + update, the shift after the last; writes cmd [7]."""
        _check(lib().storm_rollout_control(self._h, x0.data_ptr(), goal.data_ptr(), cmd.data_ptr(), int(iterations),
                                           int(bool(shift)), _stream()), "storm_rollout_control")
        return cmd

    # -- state -------------------------------------------------------------
    def get_state(self):
        mean = np.zeros((self.H, DOF), dtype=np.float32)
        sigma2 = np.zeros(self._sig_shape(), dtype=np.float32)
        step = ctypes.c_uint32()
        _check(lib().storm_rollout_get_state(self._h, mean.ctypes.data, sigma2.ctypes.data, ctypes.addressof(step),
                                             _stream()), "storm_rollout_get_state")
        return mean, sigma2, step.value

    def set_state(self, mean=None, sigma2=None, step=None):
        m = None if mean is None else np.ascontiguousarray(mean, dtype=np.float32)
        s = None if sigma2 is None else np.ascontiguousarray(sigma2, dtype=np.float32)
        st = None if step is None else ctypes.c_uint32(int(step))
        _check(lib().storm_rollout_set_state(self._h, None if m is None else m.ctypes.data,
                                             None if s is None else s.ctypes.data,
                                             None if st is None else ctypes.addressof(st), _stream()),
               "storm_rollout_set_state")

    def graph(self, x0, goal, cmd, iterations=1, shift=True, refine_iters=0, lr=0.05):
        """Capture one control step (K iterations, then optionally Adam
        refinement) into a HIP graph reading x0 / goal and writing cmd
        (device tensors whose storage must outlive the graph)."""
        if refine_iters:
            def create(h, x0p, gp, cp, it, sh, stream, out):
                return lib().storm_rollout_graph_create_refine(h, x0p, gp, cp, it, sh, int(refine_iters),
                                                               float(lr), stream, out)

            return StepGraph(self, x0, goal, cmd, iterations, shift, create=create)
        return StepGraph(self, x0, goal, cmd, iterations, shift)

    # -- differentiable form -------------------------------------------------
    def grad(self, mean, goal, x0=None, noise=None):
        """(dJ/dmu [H][7], J) of the expected horizon cost at `mean` with the
        last step's noise (or `noise` [7][N][H])."""
        x0 = self.x0 if x0 is None else x0
        g = torch.empty_like(self._mean_like)
        J = torch.empty(1, dtype=torch.float32, device=self.device)
        _check(lib().storm_rollout_grad(self._h, _ptr(x0), _ptr(goal), _ptr(mean.contiguous()), _ptr(noise),
                                        _ptr(g), _ptr(J), _stream()), "storm_rollout_grad")
        return g, J

    def refine(self, goal, iterations=3, lr=0.05, x0=None, cmd=None, shift=True):
        """Adam refinement of the stored mean, then command and shift."""
        x0 = self.x0 if x0 is None else x0
        cmd = self.cmd if cmd is None else cmd
        _check(lib().storm_rollout_refine(self._h, _ptr(x0), _ptr(goal), int(iterations), float(lr), _ptr(cmd),
                                          int(bool(shift)), _stream()), "storm_rollout_refine")
        return cmd

    def status(self):
        f = ctypes.c_uint32()
        _check(lib().storm_rollout_status(self._h, ctypes.byref(f), _stream()), "storm_rollout_status")
        return f.value


class StepGraph:
    """A captured control step; launch() enqueues it on the current stream."""

    def __init__(self, owner, x0, goal, cmd, iterations, shift, create=None):
        self.owner = owner
        self._keep = (x0, goal, cmd)
        create = lib().storm_rollout_graph_create if create is None else create
        h = ctypes.c_void_p()
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            _check(create(owner._h, _ptr(x0), _ptr(goal), _ptr(cmd), int(iterations), int(bool(shift)), _stream(),
                          ctypes.byref(h)), "graph_create")
        torch.cuda.current_stream().wait_stream(stream)
        self._h = h
        self._launch = lib().storm_rollout_graph_launch

    def launch(self, stream=None):
        code = self._launch(self._h, _stream() if stream is None else ctypes.c_void_p(stream))
        if code != STORM_OK:
            raise StormError(code, "storm_rollout_graph_launch")

    def close(self):
        if getattr(self, "_h", None) is not None and self._h.value:
            lib().storm_rollout_graph_destroy(self._h)
            self._h = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class Batch:
    """Many independent problems sharing one robot (batched form)."""

    def __init__(self, problems, device=None):
        self.device = torch.device("cuda") if device is None else torch.device(device)
        self.problems = list(problems)
        P = len(self.problems)
        self.P = P
        params = (storm_params * P)()
        scenes = (storm_scene * P)()
        self._keep = []
        for k, pr in enumerate(self.problems):
            sp, dt = make_params(pr.params)
            sc, obs = make_scene(pr.obstacles)
            params[k] = sp
            scenes[k] = sc
            self._keep += [dt, obs]
        rb, sph = make_robot(self.problems[0].spheres)
        self._keep += [rb, sph]
        h = ctypes.c_void_p()
        torch.cuda.init()
        with torch.cuda.device(self.device):
            _check(lib().storm_batch_init(ctypes.byref(h), P, params, ctypes.byref(rb), scenes, _stream()),
                   "storm_batch_init")
        self._h = h
        self.x0 = torch.tensor(np.stack([np.concatenate([pr.q0, pr.v0, pr.a0]) for pr in self.problems]),
                               dtype=torch.float32, device=self.device).contiguous()
        self.cmd = torch.zeros((P, DOF), dtype=torch.float32, device=self.device)

    def close(self):
        if getattr(self, "_h", None) is not None and self._h.value:
            lib().storm_batch_destroy(self._h)
            self._h = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def step(self, goals, x0=None):
        x0 = self.x0 if x0 is None else x0
        _check(lib().storm_batch_step(self._h, _ptr(x0), _ptr(goals), _stream()), "storm_batch_step")

    def update(self, cmd=None, shift=True):
        cmd = self.cmd if cmd is None else cmd
        _check(lib().storm_batch_update(self._h, _ptr(cmd), int(bool(shift)), _stream()), "storm_batch_update")
        return cmd

    def graph(self, x0, goals, cmd, iterations=1, shift=True, refine_iters=0, lr=0.05):
        """Capture one control step of every problem (K iterations, then
        optionally batched Adam refinement) into a HIP graph."""
        if refine_iters:
            def create(h, x0p, gp, cp, it, sh, stream, out):
                return lib().storm_batch_graph_create_refine(h, x0p, gp, cp, it, sh, int(refine_iters), float(lr),
                                                             stream, out)

            return StepGraph(self, x0, goals, cmd, iterations, shift, create=create)
        return StepGraph(self, x0, goals, cmd, iterations, shift, create=lib().storm_batch_graph_create)

    def refine(self, goals, iterations=3, lr=0.05, x0=None, cmd=None, shift=True):
        """Batched Adam refinement of every problem's stored mean (after
        update(shift=False)); returns the commands [P][7]."""
        x0 = self.x0 if x0 is None else x0
        cmd = self.cmd if cmd is None else cmd
        _check(lib().storm_batch_refine(self._h, _ptr(x0), _ptr(goals), int(iterations), float(lr), _ptr(cmd),
                                        int(bool(shift)), _stream()), "storm_batch_refine")
        return cmd

    def config(self):
        c = storm_launch_config()
        _check(lib().storm_batch_get_config(self._h, ctypes.byref(c)), "storm_batch_get_config")
        return {"waves": c.waves, "grid": c.grid, "cost_order": c.cost_order}

    def set_config(self, waves, grid, cost_order=1):
        c = storm_launch_config(int(waves), int(grid), int(cost_order))
        _check(lib().storm_batch_set_config(self._h, ctypes.byref(c)), "storm_batch_set_config")

    def autotune(self, goals, x0=None, reps=5):
        x0 = self.x0 if x0 is None else x0
        best = storm_launch_config()
        times = np.zeros(64, dtype=np.float32)
        n = ctypes.c_int32(64)
        _check(lib().storm_batch_autotune(self._h, _ptr(x0), _ptr(goals), int(reps), _stream(), ctypes.byref(best),
                                          times.ctypes.data, ctypes.byref(n)), "storm_batch_autotune")
        return {"waves": best.waves, "grid": best.grid, "cost_order": best.cost_order}, times[: n.value].copy()

    def get_state(self, p):
        pr = self.problems[p].params
        mean = np.zeros((pr.horizon, DOF), dtype=np.float32)
        sigma2 = np.zeros((pr.horizon, DOF) if getattr(pr, "cov_per_step", 0) else DOF, dtype=np.float32)
        step = ctypes.c_uint32()
        _check(lib().storm_batch_get_state(self._h, int(p), mean.ctypes.data, sigma2.ctypes.data,
                                           ctypes.addressof(step), _stream()), "storm_batch_get_state")
        return mean, sigma2, step.value

    def costs(self, p):
        C = np.zeros(self.problems[p].params.n_particles, dtype=np.float32)
        _check(lib().storm_batch_costs(self._h, int(p), C.ctypes.data, _stream()), "storm_batch_costs")
        return C


class ExpectedCost(torch.autograd.Function):
    """J(mean) = (1/N) sum_i C_i(mean + sigma eps_i) with the last step's
    noise held fixed, differentiated by the hand-written adjoint kernel.

    One adjoint launch yields both J and its gradient (the reverse pass
    recomputes the states it needs; no forward-only path is cheaper than a
    full rollout), so forward runs it and keeps the gradient, which belongs
    to the inputs of that forward call; backward only scales it by the
    incoming gradient.  A forward whose result is never differentiated still
    pays for the reverse pass."""

    @staticmethod
    def forward(ctx, mean, rollout, goal, x0=None, noise=None):
        g, J = rollout.grad(mean.detach(), goal, x0=x0, noise=noise)
        ctx.save_for_backward(g)
        return J.reshape(())

    @staticmethod
    def backward(ctx, grad_out):
        (g,) = ctx.saved_tensors
        return grad_out * g, None, None, None, None


def plant_step(x, cmd, dt):
    """Apply commands cmd [n][7] to states x [n][3][7] for dt seconds (Eq. 7)."""
    n = cmd.shape[0] if cmd.dim() == 2 else 1
    _check(lib().storm_plant_step(_ptr(x), _ptr(cmd), int(n), float(dt), _stream()), "storm_plant_step")


def fk(q, spheres=None):
    """Batched flange pose [n][12] and manipulability [n] of joint
    configurations q [n][7] (device tensor) through storm_fk, or, where q is
    as a program holds it (contiguous float32 rows of seven), storm_fk_rows."""
    n = q.shape[0]
    rows = q.dtype == torch.float32 and q.dim() == 2 and q.shape[1] == DOF and q.is_contiguous()
    qs = q if rows else q.t().contiguous()
    call = lib().storm_fk_rows if rows else lib().storm_fk
    pose = torch.empty((12, n), dtype=torch.float32, device=q.device)
    manip = torch.empty(n, dtype=torch.float32, device=q.device)
    rb, _keep = make_robot(spheres)
    _check(call(ctypes.byref(rb), _ptr(qs), int(n), _ptr(pose), _ptr(manip), _stream()), "storm_fk")
    return pose.t(), manip
