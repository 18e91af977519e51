// programs.hip -- structured programs (While / If / sequences of effects) (gfx950).
//
// Programs are independent, so one lane runs one program: the statuses of its (at most
// 64) variables are two bit planes in registers (CPU copy valid, GPU copy valid).  Every
// reduction costs one step of fuel, as in the rules While-True / While-False / IF-True /
// IF-False and Effect / Remote Effect; stuck effects are flagged and skipped.
//
// A wave first turns its 64 programs into steps in LDS (k_run_steps): one word per
// statement holding the effect as bit masks, the condition, and the two statements that
// can follow, so that running a step is straight-line code with one LDS read, the same
// for effects, While and If.  Programs too long for that, or with too little fuel, are walked in place
// (k_run_programs): their syntax tree, serialised in prefix order, with a stack of resume
// points in LDS, where entering a While body or an If branch pushes where to go when the
// block ends (the While header, which evaluates its condition again, or the word after
// the If).
#include "device.h"
#include "internal.h"
#include "prof.h"

namespace vc {

constexpr int PROG_DEPTH = 16;      // nesting levels
constexpr int PROG_BLOCK = 128;     // lanes per workgroup (LDS: resume stack per lane)

namespace {

constexpr EffectTable TABLE = make_table();

// a resume point: program-relative word offsets, 16-bit when every program is shorter
// than 2^16 words (half the LDS per lane: more waves in flight)
template <class T>
struct Frame {
    T resume, end;
};

template <class T>
__global__ __launch_bounds__(PROG_BLOCK) void k_run_programs(
    const uint64_t *__restrict__ prog_off, uint64_t n_prog, const uint32_t *__restrict__ words, uint32_t n_vars,
    const uint64_t *__restrict__ choice, const uint8_t *__restrict__ init, uint64_t fuel,
    uint64_t *__restrict__ steps_out, uint64_t *__restrict__ effects_out, uint64_t *__restrict__ stuck_out,
    uint64_t *__restrict__ first_out, uint8_t *__restrict__ done_out, uint8_t *__restrict__ final_out)
{
    __shared__ Frame<T> s_stack[PROG_DEPTH][PROG_BLOCK];
    __shared__ uint32_t s_f4[16], s_stuck[16];
    if (threadIdx.x < 16) {
        s_f4[threadIdx.x] = TABLE.f4[threadIdx.x];
        s_stuck[threadIdx.x] = TABLE.stuck[threadIdx.x];
    }
    __syncthreads();
    const uint32_t me = threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * PROG_BLOCK;
    for (uint64_t p = (uint64_t)blockIdx.x * PROG_BLOCK + me; p < n_prog; p += stride) {
        const uint64_t base = prog_off[p];
        const uint32_t len = (uint32_t)(prog_off[p + 1] - base);
        const uint32_t *w = words + base;
        uint64_t cpl = 0, gpl = 0; // bit v: CPU / GPU copy of variable v valid
        for (uint32_t v = 0; v < n_vars; v++) {
            const uint32_t s = init ? init[p * n_vars + v] : 1u;
            cpl |= (uint64_t)(s & 1u) << v;
            gpl |= (uint64_t)((s >> 1) & 1u) << v;
        }
        const uint64_t ch = choice ? choice[p] : 0ull;
        uint64_t steps = 0, effects = 0, stuck = 0, first = 0, nch = 0;
        uint32_t pc = 0, end = len, depth = 0;
        bool done = true;
        for (;;) {
            if (pc >= end) {
                if (depth == 0)
                    break;
                depth--;
                pc = s_stack[depth][me].resume;
                end = s_stack[depth][me].end;
                continue;
            }
            if (steps == fuel) {
                done = false;
                break;
            }
            steps++;
            const uint32_t word = w[pc], kind = word >> 30, x = word & 0xFFFFFFu;
            if (kind == 0) {
                const uint32_t fc = fcode((word >> 24) & 7u, (word >> 27) & 1u);
                const uint32_t s = (uint32_t)((cpl >> x) & 1u) | ((uint32_t)((gpl >> x) & 1u) << 1);
                const uint32_t bad = (s_stuck[fc] >> s) & 1u;
                const uint32_t post = fapply(s_f4[fc], s); // a stuck effect leaves s
                if (bad) {
                    if (stuck == 0)
                        first = effects;
                    stuck++;
                }
                effects++;
                const uint64_t m = 1ull << x;
                cpl = (cpl & ~m) | ((uint64_t)(post & 1u) << x);
                gpl = (gpl & ~m) | ((uint64_t)((post >> 1) & 1u) << x);
                pc++;
                continue;
            }
            // a condition: rules valid / invalid, rem-valid / rem-invalid, or the
            // program's next choice bit
            const uint32_t ck = (word >> 24) & 3u;
            bool c;
            if (ck == 0)
                c = (cpl >> x) & 1u;
            else if (ck == 1)
                c = (gpl >> x) & 1u;
            else
                c = (ch >> (nch++ & 63u)) & 1u;
            const uint32_t n = w[pc + 1];
            if (kind == 1) { // While-True enters the body, resuming at the header
                if (c) {
                    s_stack[depth][me] = Frame<T>{(T)pc, (T)end};
                    depth++;
                    end = pc + 2 + n;
                    pc = pc + 2;
                } else {
                    pc = pc + 2 + n;
                }
            } else { // IF-True / IF-False: the branch, resuming after the If
                const uint32_t m2 = w[pc + 2];
                s_stack[depth][me] = Frame<T>{(T)(pc + 3 + n + m2), (T)end};
                depth++;
                end = c ? pc + 3 + n : pc + 3 + n + m2;
                pc = c ? pc + 3 : pc + 3 + n;
            }
        }
        steps_out[p] = steps;
        effects_out[p] = effects;
        stuck_out[p] = stuck;
        first_out[p] = stuck ? first : effects;
        done_out[p] = done ? 1 : 0;
        for (uint32_t v = 0; v < n_vars; v++)
            final_out[p * n_vars + v] = (uint8_t)(((cpl >> v) & 1u) | (((gpl >> v) & 1u) << 1));
    }
}

// ----------------------------------------------------------------------------------
// programs as steps in LDS
// ----------------------------------------------------------------------------------
// A step: where its variable's status lies (bits 0-5), the copies its effect needs valid
// (6-7), the change it makes to a status s, (s & a) ^ b (a 8-9, b 10-11; statuses and
// masks as CPU | GPU << 1); its outcome (12-13: the CPU copy valid, the GPU copy valid,
// the next choice, always true); the statement that follows a true outcome (14-22) and a
// false one (23-31).  Statements are named by their first word; the program's length
// stands for its end, which has a step of its own that changes and counts nothing and
// follows itself.
constexpr uint32_t STEP_CHOICE = 2, STEP_TRUE = 3;
constexpr uint32_t STEP_MAX = 511; // longest program a step can name

__device__ __forceinline__ uint32_t make_step(uint32_t at, uint32_t need, uint32_t a, uint32_t b, uint32_t outcome,
                                              uint32_t if_true, uint32_t if_false)
{
    return at | (need << 6) | (a << 8) | (b << 10) | (outcome << 12) | (if_true << 14) | (if_false << 23);
}

// The statuses of a program's variables.  Up to 16 variables they are pairs of bits in one
// register, so that a status is one bit-field read away (a step's low 5 bits are the
// field's place); up to 32, pairs in 64 bits; up to 64, two planes.
struct Statuses16 {
    uint32_t st = 0;
    __device__ static uint32_t place(uint32_t v) { return 2u * v; }
    __device__ uint32_t get(uint32_t e) const { return __builtin_amdgcn_ubfe(st, e, 2u); }
    __device__ void change(uint32_t e, uint32_t d) { st ^= d << (e & 31u); }
};
struct Statuses32 {
    uint64_t st = 0;
    __device__ static uint32_t place(uint32_t v) { return 2u * v; }
    __device__ uint32_t get(uint32_t e) const { return (uint32_t)(st >> (e & 63u)) & 3u; }
    __device__ void change(uint32_t e, uint32_t d) { st ^= (uint64_t)d << (e & 63u); }
};
struct Statuses64 {
    uint64_t cpl = 0, gpl = 0;
    __device__ static uint32_t place(uint32_t v) { return v; }
    __device__ uint32_t get(uint32_t e) const
    {
        return ((uint32_t)(cpl >> (e & 63u)) & 1u) | (((uint32_t)(gpl >> (e & 63u)) & 1u) << 1);
    }
    __device__ void change(uint32_t e, uint32_t d)
    {
        cpl ^= (uint64_t)(d & 1u) << (e & 63u);
        gpl ^= (uint64_t)(d >> 1) << (e & 63u);
    }
};

// The statements of one program, held as its words in column `code` (one word every WAVE),
// become steps in place, in one pass in prefix order.  Blocks nest: `stack` holds the
// enclosing blocks' ends and what follows them, 16 bits each.  What follows a statement is
// the next word, or, at the end of its block, what follows the block: the While header,
// or what follows the If.
template <class ST>
__device__ __forceinline__ void compile_steps(uint32_t *code, uint32_t len, uint32_t *stack)
{
    uint32_t pc = 0, end = len, exit = len, depth = 0;
    while (pc < len) {
        while (pc == end && depth) {
            depth--;
            const uint32_t f = stack[depth * WAVE];
            end = f & 0xFFFFu;
            exit = f >> 16;
        }
        const uint32_t word = code[pc * WAVE], kind = word >> 30, x = word & 63u;
        if (kind == 0) {
            const uint32_t op = (word >> 24) & 7u, own = (word & (1u << 27)) ? 2u : 1u;
            const uint32_t next = pc + 1 == end ? exit : pc + 1;
            const uint32_t need = (op == OP_R || op == OP_PUSH) ? own : (op == OP_PULL ? own ^ 3u : 0u);
            const uint32_t set = op == OP_W ? own : ((op == OP_PUSH || op == OP_PULL) ? 3u : 0u);
            code[pc * WAVE] = make_step(ST::place(x), need, op == OP_W ? 3u : set, set, STEP_TRUE, next, next);
            pc++;
            continue;
        }
        const uint32_t ck = (word >> 24) & 3u, n = code[(pc + 1) * WAVE];
        const uint32_t m = kind == 2 ? code[(pc + 2) * WAVE] : 0u, body = pc + (kind == 2 ? 3u : 2u);
        const uint32_t after = body + n + m, next = after == end ? exit : after;
        const uint32_t back = kind == 1 ? pc : next; // what follows the body or a branch
        const uint32_t t = n ? body : back, f = m ? body + n : next;
        code[pc * WAVE] = make_step(ck == STEP_CHOICE ? 0u : ST::place(x), 0u, 0u, 0u, ck, t, f);
        if (n || m) {
            stack[depth++ * WAVE] = end | (exit << 16);
            if (n && m) // the second branch's frame lies under the first's
                stack[depth++ * WAVE] = after | (next << 16);
            end = n ? body + n : after;
            exit = back;
        }
        pc = body;
    }
    code[len * WAVE] = make_step(0u, 0u, 0u, 0u, 0u, len, len);
}

// One wave, 64 programs.  LDS columns of one word per lane (no bank is shared by two
// lanes, whatever their statements): rows [0, rows) the words and then the steps, rows
// above the nesting stack.  Reading a program's words from memory at every step bounds the
// walk in place (64 lanes on 64 cache lines, 2-3 loads a step).  Here it is the issue of
// about 33 VALU instructions a step, and the two waves per SIMD that 65 rows leave room
// for: 2^18 programs of up to 64 words over 16 variables, fuel 4096 (8.0e8 reductions),
// take 1.5 ms against 8.8 ms in place; 2^16 programs of 230 words (one wave on three of
// four SIMDs) 0.99 ms against 6.8.
template <class ST>
__global__ __launch_bounds__(WAVE) void k_run_steps(
    const uint64_t *__restrict__ prog_off, uint64_t n_prog, const uint32_t *__restrict__ words, uint32_t n_vars,
    uint32_t rows, const uint64_t *__restrict__ choice, const uint8_t *__restrict__ init, uint32_t fuel,
    uint64_t *__restrict__ steps_out, uint64_t *__restrict__ effects_out, uint64_t *__restrict__ stuck_out,
    uint64_t *__restrict__ first_out, uint8_t *__restrict__ done_out, uint8_t *__restrict__ final_out)
{
    extern __shared__ uint32_t s_col[];
    const uint32_t me = threadIdx.x;
    uint32_t *const code = s_col + me;
    const uint64_t stride = (uint64_t)gridDim.x * WAVE;
    for (uint64_t p = (uint64_t)blockIdx.x * WAVE + me; p < n_prog; p += stride) {
        const uint64_t base = prog_off[p];
        const uint32_t len = (uint32_t)(prog_off[p + 1] - base);
        const uint32_t *w = words + base;
        constexpr uint32_t BATCH = 16; // loads in flight
        for (uint32_t i = 0; i < len; i += BATCH) {
            uint32_t v[BATCH];
#pragma unroll
            for (uint32_t q = 0; q < BATCH; q++)
                v[q] = w[i + q < len ? i + q : len - 1];
#pragma unroll
            for (uint32_t q = 0; q < BATCH; q++)
                if (i + q < len)
                    code[(i + q) * WAVE] = v[q];
        }
        compile_steps<ST>(code, len, code + rows * WAVE);
        ST st;
        for (uint32_t v = 0; v < n_vars; v++)
            st.change(ST::place(v), init ? init[p * n_vars + v] & 3u : 1u);
        const uint64_t ch = choice ? choice[p] : 0ull;
        uint32_t steps = 0, effects = 0, stuck = 0, first = ~0u, nch = 0, pc = 0;
        auto step = [&] {
            const uint32_t e = code[pc * WAVE];
            const uint32_t s = st.get(e), k = (e >> 12) & 3u;
            steps += pc != len ? 1u : 0u;
            // the effect (a condition changes and needs nothing); all arithmetic, so that the
            // compiler adds no branches
            const uint32_t lack = (e >> 6) & ~s, bad = (lack | (lack >> 1)) & 1u;
            const uint32_t cand = effects | (bad - 1u);
            first = first < cand ? first : cand;
            stuck += bad;
            effects += k == STEP_TRUE ? 1u : 0u;
            st.change(e, ((s & (e >> 8)) ^ (e >> 10)) & 3u & (bad - 1u));
            // the outcome: rules valid / invalid, rem-valid / rem-invalid, or the
            // program's next choice bit
            const uint32_t bit = (uint32_t)(ch >> (nch & 63u)) & 1u;
            const uint32_t outcomes = s | (bit << STEP_CHOICE) | (1u << STEP_TRUE);
            nch += k == STEP_CHOICE ? 1u : 0u;
            pc = (e >> (((outcomes >> k) & 1u) ? 14 : 23)) & STEP_MAX;
        };
        // a program that has ended stays at its end, so the ends are looked for once every
        // UNROLL steps only
        constexpr uint32_t UNROLL = 4;
        uint32_t left = fuel;
        while (left >= UNROLL && pc != len) {
#pragma unroll
            for (uint32_t q = 0; q < UNROLL; q++)
                step();
            left -= UNROLL;
        }
        if (pc != len)
            for (; left; left--)
                step();
        steps_out[p] = steps;
        effects_out[p] = effects;
        stuck_out[p] = stuck;
        first_out[p] = stuck ? first : effects;
        done_out[p] = pc == len ? 1 : 0;
        for (uint32_t v = 0; v < n_vars; v++)
            final_out[p * n_vars + v] = (uint8_t)st.get(ST::place(v));
    }
}

} // namespace

// Whether the programs run as steps in LDS: a step names statements by 9 bits, the
// steps' counters have 32 bits, and a wave's columns (the longest program, its end and two
// nesting frames per level) fit the 64 KiB that a launch may take.
static size_t steps_lds(uint64_t longest, uint32_t depth) { return (longest + 1 + 2 * depth) * (size_t)(WAVE * 4); }
static bool fits_steps(uint64_t longest, uint32_t depth, uint64_t fuel)
{
    return longest <= STEP_MAX && steps_lds(longest, depth) <= 65536 && fuel < (1ull << 32);
}

// Whether that is worth it: a wave makes the steps of all its words first (about 0.4 us a word,
// in as many rounds as the columns leave waves on the device), and a reduction in place takes
// 1.6 us (in rounds of 4,096 waves).  Kernel times in place and by steps, by program words and
// fuel: 2^17 programs 24 / 8 21.6 and 25.1 us, 24 / 16 38 and 26, 64 / 16 43 and 49, 64 / 32 78
// and 52, 240 / 128 264 and 449, 240 / 512 931 and 594; 2^20 programs 64 / 32 334 and 317; 2,048
// programs 240 / 32 66 and 94, 240 / 128 208 and 102.
static bool worth_steps(uint64_t n_prog, uint64_t longest, uint32_t depth, uint64_t fuel)
{
    const uint64_t waves = ceil_div(n_prog, (uint64_t)WAVE), per_cu = 163840 / steps_lds(longest, depth);
    const uint64_t rounds = ceil_div(waves, 256 * (per_cu < 32 ? per_cu : 32)), in_place = ceil_div(waves, (uint64_t)4096);
    return 7 * fuel * in_place >= 2 * longest * rounds;
}

void launch_run_programs(const uint64_t *prog_off, uint64_t n_prog, const uint32_t *words, uint32_t n_vars,
                         const uint64_t *choice, const uint8_t *init, uint64_t fuel, uint64_t *steps,
                         uint64_t *effects, uint64_t *stuck, uint64_t *first, uint8_t *done, uint8_t *final_out,
                         uint64_t longest, uint32_t depth, hipStream_t s)
{
    if (!n_prog)
        return;
    if (fits_steps(longest, depth, fuel) && worth_steps(n_prog, longest, depth, fuel)) {
        const uint64_t waves = ceil_div(n_prog, (uint64_t)WAVE);
        const unsigned grid = (unsigned)(waves > 1048576 ? 1048576 : waves);
        const uint32_t rows = (uint32_t)longest + 1;
        const size_t lds = steps_lds(longest, depth);
        const auto kernel = n_vars <= 16   ? k_run_steps<Statuses16>
                            : n_vars <= 32 ? k_run_steps<Statuses32>
                                           : k_run_steps<Statuses64>;
        ProfScope p(s, "run_programs");
        kernel<<<grid, WAVE, lds, s>>>(prog_off, n_prog, words, n_vars, rows, choice, init, (uint32_t)fuel, steps,
                                       effects, stuck, first, done, final_out);
        return;
    }
    const bool short_programs = longest < (1ull << 16);
    uint64_t g = ceil_div(n_prog, PROG_BLOCK);
    const unsigned grid = (unsigned)(g > 65535 ? 65535 : g);
    ProfScope p(s, "run_programs");
    if (short_programs)
        k_run_programs<uint16_t><<<grid, PROG_BLOCK, 0, s>>>(prog_off, n_prog, words, n_vars, choice, init, fuel, steps,
                                                             effects, stuck, first, done, final_out);
    else
        k_run_programs<uint32_t><<<grid, PROG_BLOCK, 0, s>>>(prog_off, n_prog, words, n_vars, choice, init, fuel, steps,
                                                             effects, stuck, first, done, final_out);
}

} // namespace vc
