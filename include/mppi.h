/*
 * mppi.h — C ABI of the MI355X MPPI library (libmppi.so).
 *
 * One MPPI iteration, as stated in arXiv 2409.07563 (Section II-C, Algorithm 1
 * and Eq. mppi_update_rule):
 *   (a1) draw K control-noise sequences eps^k_t ~ N(0, Sigma), t < T;
 *   (a2) roll every sample out, x <- F(x, u_t + eps^k_t), and accumulate the
 *        running cost on each post-step state plus the terminal cost -> J^k;
 *   (a3) baseline rho = min_k J^k;
 *   (a4) normaliser eta = sum_k exp(-(J^k - rho) / lambda);
 *   (a5) weights w^k = exp(-(J^k - rho) / lambda) / eta;
 *   (a6) control update U_t = u_t + sum_k w^k eps^k_t;
 *   (a7) repeat with u <- U and fresh noise (the outer loop of Algorithm 1).
 *
 * Conventions
 *   - Every pointer prefixed d_ is device memory on the GPU the context was
 *     created on; every other pointer is host memory.  The caller owns all
 *     memory.  The library allocates no device memory: the caller passes one
 *     workspace (size from mppi_workspace_bytes) that must outlive the context.
 *   - Every call after mppi_create is enqueued on the context's HIP stream and
 *     returns before the GPU work finishes (stream order is the only ordering).
 *   - Arrays are binary32, row-major, densely packed unless a stride is given.
 *   - Errors: invalid arguments return MPPI_EINVAL synchronously with a message
 *     in mppi_last_error(); a failed HIP call returns MPPI_EDEVICE.  A context
 *     is not thread-safe; distinct contexts are independent.
 *   - Non-finite rollout costs count as +inf (weight 0).  If every cost of an
 *     iteration is non-finite, U is left equal to u and the status word read by
 *     mppi_get_debug(MPPI_DEBUG_STATS) is MPPI_ENUMERIC.
 */
#ifndef MPPI_H
#define MPPI_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

#define MPPI_ABI_VERSION 4u
#define MPPI_MAX_STATE 16
#define MPPI_MAX_CONTROL 8

typedef enum mppi_status {
  MPPI_OK = 0,
  MPPI_EINVAL = -1,      /* invalid argument (message in mppi_last_error) */
  MPPI_ENOMEM = -2,      /* workspace too small */
  MPPI_EDEVICE = -3,     /* a HIP runtime call failed */
  MPPI_ESTATE = -4,      /* call out of order (e.g. iterate before set_state) */
  MPPI_EUNSUPPORTED = -5,/* combination not built */
  MPPI_ENUMERIC = -6     /* every rollout cost was non-finite */
} mppi_status;

/* Dynamics F (Eq. dynamics, Section II).  State / control dimensions:
 *   DOUBLE_INTEGRATOR 4/2: (px, py, vx, vy), (ax, ay)
 *   BICYCLE           5/2: (px, py, yaw, speed, steer), (accel, steer rate);
 *                          d/dt = (s cos yaw, s sin yaw, s tan(steer)/L, a, r)
 *   QUADROTOR        13/4: p(3), q = (w,x,y,z) Hamilton, v(3) world, omega(3)
 *                          body; (thrust, tau_x, tau_y, tau_z);
 *                          q' = q (x) (0, omega)/2, v' = R(q)(0,0,F)/mass - g e3,
 *                          omega' = J^-1 (tau - omega x J omega); q is
 *                          renormalised after each step
 *   BICYCLE_MLP       5/2: bicycle step + dt * g([x_t; v_t]),
 *                          g = W3 tanh(W2 tanh(W1 z + b1) + b2) + b3,
 *                          H = 16, 32 or 64 hidden units; costs QUADRATIC and
 *                          TRACK; the MLP runs on the matrix cores in
 *                          binary32 */
typedef enum mppi_dynamics {
  MPPI_DYN_DOUBLE_INTEGRATOR = 0,
  MPPI_DYN_BICYCLE = 1,
  MPPI_DYN_QUADROTOR = 2,
  MPPI_DYN_BICYCLE_MLP = 3
} mppi_dynamics;

/* Integrator of one step with the control held: forward Euler (the paper's
 * default, Section II) or classic fourth-order Runge-Kutta. */
typedef enum mppi_integrator { MPPI_INT_EULER = 0, MPPI_INT_RK4 = 1 } mppi_integrator;

/* Running cost l(x_{t+1}, v_t) and terminal cost phi(x_T); meaning of
 * mppi_params.w[] per kind:
 *   QUADRATIC     w[0..n) = Q diag, w[8..8+m) = R diag, w[16..16+n) = Qf diag,
 *                 ref = goal (n):  l = (x-g)'Q(x-g) + v'Rv,  phi = (x-g)'Qf(x-g)
 *   PATH_CIRCLES  w = (w_lat, w_head, w_speed, v_ref, r_accel, r_steer, crash,
 *                 terminal_scale); spline y = s(x) required; circles required:
 *                 l = w_lat e^2 + w_head (yaw - atan s'(px))^2
 *                     + w_speed (speed - v_ref)^2 + r_accel a^2 + r_steer r^2
 *                     + crash * [p inside some circle],
 *                 e = py - s(px), px clamped to the knot range;
 *                 phi = terminal_scale * (the first three terms)
 *   PATH_COSTMAP  as PATH_CIRCLES with the crash term replaced by the bilinear
 *                 costmap value at p (cell centres, clamp to edge)
 *   HOVER         w = (w_p, w_v, w_w, w_q, w_u, w_box, box, terminal_scale),
 *                 ref = (waypoint 3, q_ref 4, u_hover 4):
 *                 c = w_p|p-pw|^2 + w_v|v|^2 + w_w|omega|^2 + w_q(1-<q,q_ref>^2)
 *                 l = c + w_u|v_ctrl-u_hover|^2 + w_box sum max(0,|p_i|-box)^2
 *                 phi = terminal_scale * c
 *   TRACK         w[0..n) = Q diag, w[8..8+m) = R diag, w[16] = terminal scale,
 *                 ref = reference states [(T+1)][n]:
 *                 l_t = (x - ref_{t+1})'Q(x - ref_{t+1}) + v'Rv,
 *                 phi = w[16] (x - ref_T)'Q(x - ref_T)
 *   GOAL_CIRCLES  w = (w_goal, r_accel, r_steer, crash, terminal_scale),
 *                 ref = goal (2): l = w_goal|p-goal|^2 + r_accel a^2
 *                 + r_steer r^2 + crash*[p inside some circle];
 *                 phi = terminal_scale * w_goal |p-goal|^2 */
typedef enum mppi_cost {
  MPPI_COST_QUADRATIC = 0,
  MPPI_COST_PATH_CIRCLES = 1,
  MPPI_COST_PATH_COSTMAP = 2,
  MPPI_COST_HOVER = 3,
  MPPI_COST_TRACK = 4,
  MPPI_COST_GOAL_CIRCLES = 5
} mppi_cost;

enum {
  MPPI_F_DEBUG = 1u,         /* keep per-sample crash counts (MPPI_DEBUG_CRASHES) */
  MPPI_F_ACCURATE_TRIG = 2u, /* bicycle: library sin/cos/tan instead of the hardware
                                transcendental units (the paper's own choice of
                                intrinsics for trigonometry, Sec. III-B) */
  MPPI_F_ROLLOUT_LANE = 4u,  /* force one lane per sample in the rollout */
  MPPI_F_ROLLOUT_QUAD = 8u,  /* force four lanes per sample (bicycle + RK4 only);
                                by default the time-parallel form or, where that is
                                slower or does not exist, four lanes per sample when
                                K <= 32768: see mppi_tuning) */
  MPPI_F_REQUIRES_GRAD = 16u, /* keep what mppi_backward needs: the rollout stores
                                state checkpoints every params.checkpoint_every
                                steps and a copy of the controls it used (BICYCLE
                                or BICYCLE_MLP with RK4 and the TRACK cost; not
                                for batch contexts) */
  MPPI_F_IMPORTANCE_SAMPLING = 32u,
                             /* beta = 1 of the importance-sampling weight (section
                                "MPPI-Generic's MPPI Implementation", Eq.
                                information_theoretic_weighting): every step adds
                                lambda (v_t - u_t/2)' Sigma^-1 u_t to the sample's
                                cost, which is the cost the weights are formed from
                                and mppi_get_debug(MPPI_DEBUG_COSTS) returns; needs
                                every sigma > 0.  Without it beta = 0 (Algorithm 1) */
  MPPI_F_BF16_MLP = 256u,    /* BICYCLE_MLP: the MLP's three matrix products take
                                bfloat16 operands (the weights and the layer inputs
                                z, h1, h2 rounded to nearest-even from binary32)
                                with binary32 accumulation on the matrix cores
                                (v_mfma_f32_16x16x32_bf16); biases and tanh stay
                                binary32.  Every tile form (rollout_block 64, or
                                the MLP split over 2 or 4 waves).  With
                                MPPI_F_REQUIRES_GRAD the adjoint
                                differentiates this forward with the roundings
                                taken as the identity (the products' derivatives
                                use the rounded weights and inputs).  Without it
                                the products are binary32 */
  MPPI_F_MEAN_SAMPLE = 128u, /* sample 0 is drawn without noise (eps_0 = 0, v = u: the
                                mean itself is one of the samples; section
                                "Sampling Distributions") */
  MPPI_F_STEP_SIZE = 64u,    /* use config.step_size as the step size gamma >= 0 of
                                the dynamic mirror-descent update (section
                                "Comparisons to sampling-efficient algorithms"):
                                U = (1 - gamma) u + gamma sum_k w_k v_k, computed as
                                u + gamma sum_k w_k eps_k; mppi_backward scales its
                                gradient to match.  Without it gamma = 1 */
};

typedef struct mppi_config {
  uint32_t abi_version;  /* must equal MPPI_ABI_VERSION */
  uint32_t dynamics;     /* mppi_dynamics */
  uint32_t integrator;   /* mppi_integrator */
  uint32_t cost;         /* mppi_cost */
  int32_t num_samples;   /* K >= 1 */
  int32_t horizon;       /* T >= 1 */
  int32_t state_dim;     /* must match the dynamics */
  int32_t control_dim;   /* must match the dynamics */
  float dt;              /* > 0 */
  float lambda;          /* temperature, > 0 */
  float sigma[MPPI_MAX_CONTROL]; /* noise std per control, >= 0 (diagonal Sigma) */
  uint64_t seed;         /* Philox key */
  uint32_t instance;     /* Philox counter word 3 (independent streams) */
  uint32_t flags;        /* MPPI_F_* */
  float step_size;       /* gamma, read only with MPPI_F_STEP_SIZE: finite, >= 0 */
  float zero_mean_fraction; /* in [0, 1]: the last floor(fraction K) samples (at
                               most K - 1 with MPPI_F_MEAN_SAMPLE) are drawn around
                               zero instead of u: v_k = eps_k, the update is
                               U = u + gamma sum_k w_k (v_k - u), their
                               importance-sampling term is zero (section
                               "Sampling Distributions").  Not with
                               MPPI_F_REQUIRES_GRAD */
} mppi_config;

/* Model and cost constants.  Every array pointer is host memory, read during
 * mppi_create only (copied into the workspace). */
typedef struct mppi_params {
  float wheelbase;        /* BICYCLE*, L > 0 */
  float mass;             /* QUADROTOR, > 0 */
  float inertia[3];       /* QUADROTOR, diagonal of J, > 0 */
  float gravity;          /* QUADROTOR */
  int32_t mlp_hidden;     /* BICYCLE_MLP: H in [1, 256] */
  const float* mlp;       /* W1[H][7] b1[H] W2[H][H] b2[H] W3[5][H] b3[5] */
  float w[32];            /* cost weights, see mppi_cost */
  const float* ref;       /* goal / waypoint data / reference trajectory */
  int32_t ref_len;        /* number of floats at ref */
  int32_t num_segments;   /* spline segments S >= 1 (PATH_*) */
  const float* knots;     /* S+1 increasing abscissae */
  const float* coef;      /* [S][4]: y = c0 + c1 d + c2 d^2 + c3 d^3, d = x - knot */
  int32_t num_circles;    /* circles (PATH_CIRCLES, GOAL_CIRCLES), may be 0 */
  const float* cx;        /* centres x [N] */
  const float* cy;        /* centres y [N] */
  const float* r2;        /* squared radii [N] */
  int32_t map_w, map_h;   /* costmap cells (PATH_COSTMAP), each >= 2 */
  float map_x0, map_y0;   /* lower-left corner of cell (0, 0) */
  float map_res;          /* cell size > 0 */
  const float* costmap;   /* [map_h][map_w] */
  int32_t checkpoint_every; /* MPPI_F_REQUIRES_GRAD: steps between state
                               checkpoints, 1..64 (0 = 10) */
  int32_t tape_len;       /* MPPI_F_REQUIRES_GRAD: updates mppi_backward_iters can
                             differentiate through, 1..1024 (0 = 16) */
  const float* sigma_t;   /* optional [T][m]: a noise standard deviation per step and
                             control (>= 0, > 0 with MPPI_F_IMPORTANCE_SAMPLING),
                             replacing config.sigma; eps = sigma_t[t][j] z (one
                             binary32 product; section "Sampling Distributions") */
  int32_t cost_cosines;   /* 0..65536 nested cosines evaluated ahead of every running
                             cost and scaled by zero: the synthetic cost-complexity
                             load of the paper's Results section.  It changes no
                             result, only the cost's computation time */
} mppi_params;

typedef struct mppi_ctx mppi_ctx;

/* Bytes of device workspace a context with this configuration needs
 * (0 if the configuration is invalid; see mppi_last_error). */
size_t mppi_workspace_bytes(const mppi_config* cfg, const mppi_params* params);

/* Create a context: the fixed inputs of Algorithm 1 (the dynamics F, the
 * running and terminal costs, the horizon T, the sample count K, the
 * temperature lambda and the noise covariance Sigma; the number of
 * iterations is mppi_iterate's argument).  d_workspace: device memory of at
 * least mppi_workspace_bytes, 256-byte aligned, owned by the caller and used
 * exclusively by this context until mppi_destroy.  hip_stream: a hipStream_t
 * (NULL = the null stream).  Copies the parameter arrays to the device and
 * waits for the copies.  The nominal controls start at zero and the iteration
 * counter at 0. */
mppi_status mppi_create(const mppi_config* cfg, const mppi_params* params,
                        void* d_workspace, size_t workspace_bytes, void* hip_stream,
                        mppi_ctx** out);

/* ---- a context that allocates nothing --------------------------------------
 * For callers that cannot allocate device memory: code under HIP graph
 * capture, tight serving loops, harnesses that forbid hipMalloc.  As
 * mppi_create for one instance, but the workspace is a fixed array of
 * MPPI_STATIC_WORKSPACE_BYTES that libmppi.so holds on every GPU it runs on
 * (each GPU its own copy) until the process ends; the call and the context's
 * later calls allocate no device memory (no hipMalloc, hipFree or allocating
 * library routine).  The context uses the current device; hip_stream, if not
 * NULL, must belong to it.  The array keeps the previous context's contents:
 * creation initialises everything an iteration reads before writing it, as
 * mppi_create does for a fresh workspace.  Every context created here on one
 * GPU shares that GPU's array, so work of two such contexts overlapping in
 * time would race: one lives per GPU at a time (a second call on the device
 * returns MPPI_ESTATE until the first is destroyed), and mppi_destroy of such
 * a context waits for its stream before it frees the array for the next one.
 * Errors: as mppi_create; MPPI_ENOMEM when mppi_workspace_bytes exceeds
 * MPPI_STATIC_WORKSPACE_BYTES (the message gives both sizes); MPPI_ESTATE as
 * above; MPPI_EINVAL for a stream of another device. */
#define MPPI_STATIC_WORKSPACE_BYTES ((size_t)64 << 20)
mppi_status mppi_create_static(const mppi_config* cfg, const mppi_params* params,
                               void* hip_stream, mppi_ctx** out);

/* ---- batches (spec extension: many independent instances) ----------
 * A batch context holds n independent MPPI instances that share dynamics,
 * integrator, cost kind and flags but each have their own K, T, dt, lambda,
 * sigma, seed / instance word and parameter arrays (their own obstacles,
 * goal, weights).  Every phase of an iteration runs all instances in one
 * launch over a work list (instance, block of samples) ordered by horizon,
 * longest first.  All calls below accept batch contexts; wherever a call
 * takes or returns a per-instance array, a batch context uses the
 * concatenation of the instances' arrays in instance order ("packed"), at
 * the offsets mppi_offsets reports.  A context from mppi_create is a batch of
 * one. */
size_t mppi_batch_workspace_bytes(const mppi_config* cfgs, const mppi_params* params, int32_t n);
mppi_status mppi_create_batch(const mppi_config* cfgs, const mppi_params* params, int32_t n,
                              void* d_workspace, size_t workspace_bytes, void* hip_stream,
                              mppi_ctx** out);
int32_t mppi_num_instances(const mppi_ctx* ctx);
enum {
  MPPI_PACKED_STATE = 0,    /* state_dim floats per instance */
  MPPI_PACKED_CONTROLS = 1, /* T*m floats per instance */
  MPPI_PACKED_SAMPLES = 2,  /* K values per instance (costs, weights, crash counts) */
  MPPI_PACKED_NOISE = 3     /* T*m*K floats per instance */
};
/* host_offsets[0..n]: element offsets of each instance in a packed array of
 * the given kind (host_offsets[n] = total length). */
mppi_status mppi_offsets(const mppi_ctx* ctx, int32_t what, int64_t* host_offsets);

/* ---- launch shapes and the autotuner (spec extension) ------------------
 * How the kernels of a context are launched; none of it changes results
 * except lanes_per_sample and rollout_form, which select a different (equally
 * accurate) rollout kernel, and update_form, which rounds the update's sums in
 * another order.  The paper picks between its kernels by timing
 * them (section "Choosing between the Split and Combined Kernels");
 * mppi_autotune does the same over this table.
 *
 * The split form (section "Split Kernel Description") runs step (a2) as two
 * kernels: the dynamics kernel integrates every sample over the horizon and
 * writes its states x_1..x_T to a trajectory buffer in the workspace; the
 * cost kernel then evaluates the running costs of all T steps in parallel
 * (cost_waves waves per 64 samples, wave g taking the steps t = g,
 * g + cost_waves, ...) and sums them per sample in a fixed order.  It exists
 * for single contexts with DOUBLE_INTEGRATOR, BICYCLE or QUADROTOR dynamics
 * (not for MLP dynamics, gradient mode or batches). */
/* The scan form runs step (a2) for the bicycle with RK4 time-parallel: with
 * the control held over a step, speed and steer advance by dt times the
 * controls, the stage yaw rates depend only on speed and steer, and the
 * position increments only on the yaw and those, so a rollout is three
 * prefix sums over time (a sample's horizon spread over 16 lanes, chunks of
 * ceil(T / 16) steps per lane) followed by the running costs of all steps in
 * parallel.  It exists for single contexts with BICYCLE dynamics, RK4 and
 * T <= 256 (not for gradient mode), with lanes_per_sample 16 and
 * rollout_block threads per workgroup.  Equally accurate: the positions are
 * summed with compensation; only the rounding order differs.
 * A context for which the form exists and neither MPPI_F_ROLLOUT_LANE nor _QUAD
 * is set is created with lanes_per_sample 0 where it is the faster one (all but
 * short horizons with many samples, and costs without circles or a two-valued
 * costmap for many samples): it runs this form with 16 or 32 lanes and 256 threads
 * until other lanes_per_sample are set, whatever the other fields. */
enum { MPPI_ROLLOUT_FUSED = 0, MPPI_ROLLOUT_SPLIT = 1, MPPI_ROLLOUT_SCAN = 2 };
/* Steps (a3)-(a6) (Algorithm 1, Eq. mppi_update_rule):
 *  TWO_PASS: a weights step in one workgroup writes the weights, then one
 *    workgroup per row forms the weighted noise sum (every context; the
 *    default for batches and gradient mode, whose adjoint reads the weights);
 *  ONE_PASS: one launch in which every row's workgroup computes the baseline,
 *    the weights and the normaliser itself from the costs (single contexts
 *    with at most 16384 samples, no gradient mode; the default there);
 *  CHUNKED: the weights step spread over workgroups of 2048 samples, each
 *    weighting its samples against its own minimum, and the rows rescale the
 *    chunks to the global minimum (single contexts, no gradient mode; the
 *    default above 16384 samples).
 * All three are equally accurate; their sums are rounded in different orders
 * (CHUNKED's weights are products of two exponentials). */
enum { MPPI_UPDATE_TWO_PASS = 0, MPPI_UPDATE_ONE_PASS = 1, MPPI_UPDATE_CHUNKED = 2 };
/* How mppi_iterate runs an iteration of a batch context:
 *  PHASES: four launches (noise, rollout, weights, update rows), each over
 *    all instances;
 *  ONE_LAUNCH: one launch per iteration with a workgroup per tile of 256
 *    samples (tiles ordered longest horizon first).  A tile draws its own
 *    noise (stored to the noise buffer), rolls out, weights its samples
 *    against its own minimum cost and forms its weighted noise rows; the
 *    workgroup that completes an instance's last tile (a per-instance
 *    completion counter) rescales the tiles to the instance's minimum and
 *    updates u, the statistics and the iteration word.  No workgroup waits
 *    for another and there is no grid-wide barrier.  Needs batch_tile 256, the
 *    two-pass update setting, at most 65536 samples per instance and a kernel
 *    for the combination (the models and costs of the per-phase kernels with
 *    two or four controls).  Noise and costs are bitwise those of PHASES; the
 *    update equals it up to the rounding order of its sums (the chunked
 *    update's arithmetic with tiles for chunks).
 * The staged calls (mppi_sample, mppi_rollout, mppi_update) always run the
 * per-phase launches. */
enum { MPPI_BATCH_PHASES = 0, MPPI_BATCH_ONE_LAUNCH = 1 };
typedef struct mppi_tuning {
  int32_t lanes_per_sample; /* rollout: 1, or 4, 8 or 16 (the bicycle with RK4, single
                               instance: RK4 stages across a quad, the running cost
                               shared by the lanes; 16 also in the scan form: the
                               horizon across the lanes); 16 for MLP dynamics and
                               gradient mode (fixed); 0 in the fused form, for a
                               context created so: the time-parallel form as above,
                               rollout_block then being without effect */
  int32_t rollout_block;    /* threads per rollout workgroup: 64, 128 or 256; for MLP
                               dynamics and gradient mode 64 (one wave per 16-sample
                               tile), or 128 / 256 (the tile's MLP split over 2
                               waves, H = 32 and 64, or 4 waves, H = 64, beside
                               the waves of the bicycle and the cost; H / 16 waves,
                               the default, only as far as that is the faster form
                               for the number of samples, else one wave) */
  int32_t batch_tile;       /* samples per work tile of a batch context: 64, 128 or 256 */
  int32_t noise_calls;      /* Philox calls per thread and sample of the
                               single-instance noise kernel: 1, 2 or 4 */
  int32_t rollout_form;     /* MPPI_ROLLOUT_FUSED (default), MPPI_ROLLOUT_SPLIT or
                               MPPI_ROLLOUT_SCAN; in the split form
                               lanes_per_sample (1, or 4 for the bicycle with RK4)
                               and rollout_block shape the dynamics kernel, in the
                               scan form lanes_per_sample is 16 or 32 */
  int32_t cost_waves;       /* split form: waves that share the steps of 64 samples in
                               the cost kernel, a power of two from 1 to 128 (up to
                               16 in one workgroup; beyond, chunks of 16 waves whose
                               partial sums a small kernel adds; default 8) */
  int32_t update_form;      /* MPPI_UPDATE_TWO_PASS, _ONE_PASS or _CHUNKED (defaults
                               as listed above) */
  int32_t batch_form;       /* batch contexts: MPPI_BATCH_PHASES or
                               MPPI_BATCH_ONE_LAUNCH (single contexts: PHASES) */
  int32_t adjoint_tiles;    /* gradient mode: mppi_backward sweeps the checkpoint
                               segments in parallel (the costate chained through each
                               segment's linear map) when the samples of nonzero
                               weight fill at most this many 16-sample tiles, else
                               one sweep per tile over the whole horizon; 0 to 128
                               (0: always the per-tile sweep; default 64; also at
                               most 1280 / units, a unit being up to 5 steps of
                               a checkpoint segment) */
} mppi_tuning;

/* The context's current launch shapes. */
mppi_status mppi_get_tuning(const mppi_ctx* ctx, mppi_tuning* out);
/* Apply launch shapes (EINVAL for a value outside its set; EUNSUPPORTED for
 * lanes_per_sample 4, 8 or 16 where no such kernel exists, or the split form
 * where it does not exist).  Rebuilds a batch's work
 * list (waits for the upload); captured iteration graphs are rebuilt on their
 * next use. */
mppi_status mppi_set_tuning(mppi_ctx* ctx, const mppi_tuning* t);
/* Time every candidate launch shape of the sampling and rollout phases on this
 * context (reps launches each, HIP events on the context's stream, after one
 * warm-up launch) and apply the fastest.  Needs mppi_set_state; overwrites the
 * noise and cost buffers (not u or the iteration word).  host_report
 * (optional, report_len bytes): one line per candidate, "phase shape time_us".
 * Synchronises the context's stream. */
mppi_status mppi_autotune(mppi_ctx* ctx, int32_t reps, char* host_report, size_t report_len);

/* x0 <- d_x0[0..n): the initial state every rollout of Algorithm 1 starts
 * from (enqueued device copy; packed for a batch).  Errors: EINVAL (NULL). */
mppi_status mppi_set_state(mppi_ctx* ctx, const float* d_x0);
/* u <- d_u[T][m] (enqueued device copy; warm start or restore; packed). */
mppi_status mppi_set_controls(mppi_ctx* ctx, const float* d_u);
/* Philox iteration word of the next sampling step (enqueued; every instance
 * of a batch). */
mppi_status mppi_set_iteration(mppi_ctx* ctx, uint32_t iteration);
/* MPC warm start between control calls (section "Beginner": a new MPC
 * iteration samples around the previous sequence moved forward by the
 * optimisation stride): u[t] <- u[t + steps] for t + steps < T, the steps past
 * the horizon take u[T-1] (fill = MPPI_SHIFT_HOLD) or 0 (MPPI_SHIFT_ZERO).
 * steps >= 0 (steps >= T leaves no old entry).  Enqueued kernel (may be
 * captured in a graph); every instance of a batch.  Errors: EINVAL. */
enum { MPPI_SHIFT_HOLD = 0, MPPI_SHIFT_ZERO = 1 };
mppi_status mppi_shift(mppi_ctx* ctx, int32_t steps, int32_t fill);

/* Staged iteration (Algorithm 1 split at its natural boundaries):
 *   mppi_sample  - (a1) eps for the current iteration word
 *   mppi_rollout - (a2) J^k from x0, u and eps
 *   mppi_update  - (a3..a6) rho, eta, w and u <- u + sum_k w^k eps^k; then the
 *                  iteration word advances by one.
 * mppi_set_costs replaces J (K floats, device) between rollout and update. */
mppi_status mppi_sample(mppi_ctx* ctx);
mppi_status mppi_rollout(mppi_ctx* ctx);
mppi_status mppi_set_costs(mppi_ctx* ctx, const float* d_costs);
mppi_status mppi_update(mppi_ctx* ctx);

/* (a7) num_iters >= 1 full iterations, warm-started (u <- U between them).
 * For num_iters >= 2 the launch sequence is captured into a hipGraph on
 * first use and replayed afterwards (the context's stream must not be under
 * capture by the caller at that first call); a single iteration (one to four
 * kernel launches) is launched directly, which reaches the GPU sooner.
 * Results are those of num_iters x (sample, rollout, update); the noise
 * visible afterwards (MPPI_DEBUG_NOISE, mppi_backward) is the last
 * iteration's.  A single context whose noise buffer is at most 64 MiB keeps a
 * second one: each iteration's noise is drawn by a launch of the iteration
 * before, and the last iteration draws the noise of the next call's first
 * one, which that call then uses unless mppi_set_iteration, mppi_sample,
 * mppi_rollout, mppi_set_costs, mppi_update, mppi_set_tuning, mppi_autotune,
 * mppi_set_theta or mppi_backward_iters came in between (mppi_set_state,
 * mppi_set_controls and mppi_shift keep it).  The noise is the same either
 * way: it depends on the seed, the iteration word and the instance only. */
mppi_status mppi_iterate(mppi_ctx* ctx, int32_t num_iters);

/* d_U[T][m] <- the current nominal control sequence, Algorithm 1's output
 * after its last update (enqueued device copy; packed for a batch).  Errors:
 * EINVAL (NULL). */
mppi_status mppi_get_controls(mppi_ctx* ctx, float* d_U);

/* ---- ordering with the caller's streams -----------------------------------
 * For callers whose tensors live on other streams than the context's (one event
 * each way, kept by the context; nothing waits on the host).  hip_stream is a
 * stream of the context's device, which need not be the current one; NULL is that
 * device's null stream:
 *   mppi_wait_stream    what the context is given from now on starts after
 *                       everything hip_stream holds now;
 *   mppi_release_stream what hip_stream is given from now on starts after
 *                       everything the context has been given.
 * Errors: EINVAL (NULL ctx), EDEVICE. */
mppi_status mppi_wait_stream(mppi_ctx* ctx, void* hip_stream);
mppi_status mppi_release_stream(mppi_ctx* ctx, void* hip_stream);
/* mppi_set_state, mppi_set_controls or mppi_set_costs (what: MPPI_PACKED_STATE,
 * MPPI_PACKED_CONTROLS or MPPI_PACKED_SAMPLES), the array read on hip_stream: it
 * starts after what hip_stream and the context hold now, what the context is given
 * from now on starts after it, and what hip_stream is given from now on may write
 * or free d_src.  Neither stream under capture.  Errors: EINVAL (NULL, unknown
 * array), EDEVICE. */
mppi_status mppi_put(mppi_ctx* ctx, int32_t what, const float* d_src, void* hip_stream);

enum {
  MPPI_DEBUG_NOISE = 0,   /* float eps[T][m][K] of the last sampling */
  MPPI_DEBUG_COSTS = 1,   /* float J[K] of the last rollout (or set_costs) */
  MPPI_DEBUG_WEIGHTS = 2, /* float w[K] of the last update */
  MPPI_DEBUG_STATS = 3,   /* float[8] per instance: rho, eta, free energy
                             rho - lambda ln(eta/K), 1/sum w^2, then the int32
                             status word (MPPI_OK / MPPI_ENUMERIC) and the int32
                             iteration word, then two zero words */
  MPPI_DEBUG_CRASHES = 4  /* int32 crashed-step count per sample [K]
                             (needs MPPI_F_DEBUG and a circles cost) */
};
/* Enqueue a device copy of an internal buffer to d_dst. */
mppi_status mppi_get_debug(mppi_ctx* ctx, int32_t what, void* d_dst);

/* ---- differentiation (spec extension) --------------------------------
 * The parameter vector theta, "gradient layout", n_theta floats:
 *   [W1 (H*7) | b1 (H) | W2 (H*H) | b2 (H) | W3 (5*H) | b3 (5)]  (BICYCLE_MLP only)
 *   [Q diag = w[0..n) of the TRACK cost (n) | wheelbase (1)].
 * mppi_theta_len: n_theta of a context (0 and an error message if the
 * context cannot differentiate). */
int32_t mppi_theta_len(const mppi_ctx* ctx);

/* Replace theta (host memory, n_theta floats in the gradient layout): the MLP
 * weights, the Q diagonal and the wheelbase.  Waits for the upload; iteration
 * graphs captured before are rebuilt on their next use.  Needs
 * MPPI_F_REQUIRES_GRAD.  Errors: EINVAL (NULL, non-finite values, wheelbase
 * <= 0), ESTATE (context without MPPI_F_REQUIRES_GRAD). */
mppi_status mppi_set_theta(mppi_ctx* ctx, const float* host_theta);

/* Gradient of a loss L on the controls U produced by the last update,
 * U = u + sum_k w_k eps_k (Algorithm 1; the nominal u of that iteration is
 * held fixed): d_grad[n_theta] <- dL/dtheta (device, gradient layout) given
 * d_dL_dU[T][m] = dL/dU (device).  Differentiates through the softmin weights
 * (w_k depends on theta only through the costs J_k; the baseline rho drops
 * out) and through every rollout: the costate is swept backwards over the
 * discrete step (the four RK4 stages and the MLP residual) from state
 * checkpoints.  Samples of weight exactly zero contribute nothing and are
 * skipped.  With few samples of nonzero weight (tuning adjoint_tiles) the
 * checkpoint segments are swept in parallel: each segment's costate map
 * (the product of its step Jacobians, formed in forward mode, and its running
 * costs' share) chains the costate across segments, so the latency is that
 * of one segment instead of the whole horizon; the result agrees with the
 * per-tile sweep up to rounding.  Binary32 throughout except the normaliser
 * eta (binary64).  Enqueued on the context's stream; the result is bitwise
 * reproducible for a given tuning.
 * Errors: EINVAL (NULL), ESTATE (no MPPI_F_REQUIRES_GRAD, or no update since
 * the last mppi_sample / mppi_rollout / mppi_set_costs), EDEVICE. */
mppi_status mppi_backward(mppi_ctx* ctx, const float* d_dL_dU, float* d_grad);

/* Gradient through every update since the tape started (the warm-started
 * iterations of Algorithm 1's outer loop): with u_{i+1} = u_i + gamma
 * sum_k w_k(u_i, theta) eps_k for i = 0..n-1 and d_dL_dU = dL/du_n (device,
 * [T][m]), d_grad[n_theta] <- dL/dtheta (device) and, if d_dL_du0 is given,
 * d_dL_du0[T][m] <- dL/du_0 (device).  In gradient mode each update records
 * its u and Philox iteration word on the tape (params.tape_len slots); the
 * tape starts over at mppi_create, mppi_set_state, mppi_set_controls,
 * mppi_set_theta and mppi_shift.  The reverse pass runs the updates
 * backwards: it rebuilds update i (its noise from the recorded word, the
 * checkpointing rollout from the recorded u_i, the weights; the last update
 * is taken from the buffers when mppi_backward could run), adds the
 * gradient of that iteration at fixed u_i, and carries dL/du_i = dL/du_{i+1} +
 * sum_k a_k dJ_k/du_i (the costs depend on u_i through v = u_i + eps and,
 * with MPPI_F_IMPORTANCE_SAMPLING, directly) to the next one.  With one
 * update it gives mppi_backward's gradient.  Synchronises the context's stream
 * once (to read the tape's length); afterwards the noise, cost and weight
 * buffers hold the first taped update's values (mppi_backward then needs a new
 * iteration).  Errors: EINVAL (NULL), ESTATE (no MPPI_F_REQUIRES_GRAD; no
 * update since the tape started; more than tape_len updates; an update whose
 * costs came from mppi_set_costs), EDEVICE. */
mppi_status mppi_backward_iters(mppi_ctx* ctx, const float* d_dL_dU, float* d_grad,
                                float* d_dL_du0);

void mppi_destroy(mppi_ctx* ctx);

/* Message of the last error on this thread; never NULL. */
const char* mppi_last_error(void);

/* ---- stand-alone noise (the same definition mppi_sample uses) ----------
 * eps[t][j][k] (row stride ldk >= K floats) of the noise definition:
 *   normal n = t*m + j of sample k comes from Philox4x32-10 (Salmon et al.,
 *   SC'11) with counter (n/4, k, iteration, instance) and key (seed lo, seed
 *   hi); slot n%4 takes the Box-Muller pair (x0,x1) or (x2,x3) and its cosine
 *   (even) or sine (odd) branch with u1 = ((a>>8)+1) 2^-24, u2 = (b>>8) 2^-24;
 *   eps = sigma_j * sqrt(-2 ln u1) * {cos,sin}(2 pi u2), where -2 ln u1 and
 *   sincos use exact range reductions and fixed binary32 polynomials
 *   (paper_2409_07563_amd/csrc/noise.h spells out every operation), so any
 *   IEEE-754 host can reproduce eps bit for bit.  sigma: host, m floats. */
mppi_status mppi_noise(uint64_t seed, uint32_t iteration, uint32_t instance, int32_t K,
                       int32_t T, int32_t m, const float* sigma, float* d_eps,
                       int64_t ldk, void* hip_stream);

/* The Box-Muller factors for every possible input (2^24 each, device):
 * d_r[j1-1] = sqrt(-2 ln(j1 2^-24)), d_c[j2] = cos(2 pi j2 2^-24),
 * d_s[j2] = sin(2 pi j2 2^-24).  For exhaustive checks of the recipe. */
mppi_status mppi_noise_tables(float* d_r, float* d_c, float* d_s, void* hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* MPPI_H */
